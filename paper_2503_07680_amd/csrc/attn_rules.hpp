// Which kernels an attention call launches: plain host functions of sizes, without HIP, so that a test without a GPU can
// ask them too.
#pragma once
#include <stdint.h>

namespace hbp {

constexpr int kNumXcd = 8;   // accelerator dies, each with its own L2
constexpr int kNumCU = 256;  // MI355X: 8 dies x 32 compute units

// A kernel whose items all fit on the chip at once gets one workgroup an item and no queue: every item starts
// at once whatever its order, and the launch that resets the counters (5 us of the stream's time) and the
// atomic in front of an item fall away.  Training step of a 1024-token pack with 4 heads of 64: 46.0 -> 36.6 us;
// of 5497 tokens with 8 heads: 119 -> 110.  The forward goes further (fwd_way).  Profile records are one per resident
// workgroup, so a call that asks for them keeps the queues.
inline bool direct_items(int64_t n_items, int64_t resident, bool records) { return !records && n_items <= resident; }

// In how many parts the `units` schedulable units of a kv head (query heads, or pairs of them) are
// dealt out: the smallest divisor of units that gives every die a queue, else units itself.
inline int heads_split(int n_kv_heads, int units) {
  for (int s = 1; s <= units; ++s)
    if (units % s == 0 && n_kv_heads * s >= 8) return s;
  return units;
}

struct PackShape {
  int d_qk, T, n_samples, Hq, Hkv;
  int g() const { return Hq / Hkv; }
  double mean_len() const { return (double)T / (n_samples > 0 ? n_samples : 1); }
};

// Launches of few rounds: one workgroup an item, dispatched by the hardware in the worklist's order (kDirect), without the
// launch that resets the queues' counters (5 us) and without the hand-over between items; and for even groups of heads
// also one head a workgroup of four wavefronts, two workgroups a compute unit, instead of a pair of heads on one K/V
// stream (kSingles): a workgroup's prologue and end are then covered by the other one, and the last round is finer.  With
// more rounds the queues balance better, and long samples need the shared stream.  `rounds`: items (pairs of heads, or
// 256-row tiles) to a compute unit; `len`: tokens a sample.  Forward, time with queues and pairs / this way, T = 2048 to
// 32768, 3 to 64 heads:
//   even, d = 64     singles, to 7: 1.03 to 1.37; to 10, samples of 100 to 250: 1.10 to 1.14
//   even, d >= 128   singles, to 2: 1.03 to 1.34; samples to 100, to 8: 1.04 to 1.23
//     kv heads dealt evenly to the dies: pairs, 2 to 4.8: 1.00 to 1.12 (samples of 1600: .98), 5.3: .99; singles there
//                    gain up to .03 more, but .96 to .99 with a sample of half the pack
//     else           pairs, 2 to 2.7: 1.00 to 1.10; 3.1: .98; singles, 2.5: .98 to 1.03
//   odd              256-row tiles, to 3.5: 1.00 to 1.52; 3.6: .99; 4.2 to 4.7: .97 to 1.03; samples to 128, 4.0 to 5.5:
//                    1.04 to 1.14
//   odd, kHalves     a workgroup of four wavefronts takes half of a 256-row tile: the longest item's chain of key tiles runs
//                    without a second wavefront on its SIMD.  Against 256-row tiles, mixed samples and one of .4 or .5:
//     d = 64         to 4.2: 1.00 to 1.31; 4.5: .97 to 1.09; len to 320, to 7.5: 1.01 to 1.24
//     d = 128        to .75: 1.02 to 1.23; .8 to 2: .93 to 1.17; len to 350, to 9: 1.02 to 1.42; 11 to 22: .95 to 1.10
//     d = 192        to 2.3: 1.01 to 1.21; 3 to 4.5: .97 to 1.13; len to 350, to 6: 1.01 to 1.20; 7.4: .99
//     len to 100     from 1.05 on: 1.10 to 1.45, and packs of that mean with a long sample .97 to 1.02 to T = 16384; with a
//                    round or less: .97 to 1.03
// The host knows the samples' mean length alone, and beyond two rounds a very long sample beside short ones loses by every
// way but the queues: 9500 tokens with a sample of 7125, 16/8 heads of 128: .96.  kDirect and kSingles therefore end at
// T = 8192 or 16384.  kHalves does not: beyond 2.5 rounds, T = 18000 to 48000, against 256-row tiles with queues, without a
// long sample / with one of .3 / of .4 or .5 / of .65 or .7 of the pack
//   d = 64, 8 heads          1.05 to 1.31 / 1.04 to 1.28 / .96 to 1.23 / .95 to 1.06
//           4                1.14 to 1.33 / 1.17 to 1.28 / 1.03 to 1.26 / .95 to 1.19
//           6/2              1.06 to 1.37 / 1.02 to 1.28 / .92 to 1.23 / .93 to 1.20
//   d = 128, 8, 12, 16 heads 1.03 to 1.23 / .95 to 1.13 / .95 to 1.06 / .96 to .98 (the losses from 4.5 rounds on)
//            9/3             1.13 to 1.23 / 1.09 to 1.15 / 1.08 to 1.21 / not measured
//   d = 192, 12/4            1.11 and 1.12 / 1.05 / 1.03 / not measured
// A bound on T there would lose the first two columns for what the last two lose.
enum FwdWay { kQueues, kDirect, kSingles, kHalves };
inline FwdWay fwd_way(const PackShape& p, int64_t n_items, bool records) {
  if (records) return kQueues;  // records are one per resident workgroup
  const int d_qk = p.d_qk, g = p.g();
  const double rounds = (double)n_items / kNumCU, len = p.mean_len();
  if (g % 2 && rounds <= 300) {
    if (len <= 100) {
      if (rounds > 1.05 && p.T <= 16384) return kHalves;
    } else if (d_qk == 64 ? rounds <= 4.2 || (len <= 320 && rounds <= 7.5)
                          : d_qk == 128 ? rounds <= 0.75 || (len <= 350 && rounds <= 9)
                                        : rounds <= 2.3 || (len <= 350 && rounds <= 6)) {
      return kHalves;
    }
  }
  if (rounds <= 2) return kSingles;
  if (p.T > (g % 2 || d_qk == 64 ? 16384 : 8192)) return kQueues;
  if (g % 2) return rounds <= 3.5 || (len <= 128 && rounds <= 5.5) ? kDirect : kQueues;
  if (d_qk == 64) return rounds <= 7 || (len <= 300 && rounds <= 10) ? kSingles : kQueues;
  if (len <= 100 && rounds <= 8) return kSingles;
  if (p.Hkv % kNumXcd) return rounds <= 2.7 ? kDirect : kQueues;
  return rounds <= 4.8 ? kDirect : kQueues;
}
// The launch: fwd_kernel<., ., HP, TP> with queues or one workgroup an item.  tile_rows: rows per query tile of the
// worklist, 128 or (odd group sizes only) 256.
struct FwdLaunch {
  int hp, tp;
  bool direct, halves;
};
inline FwdLaunch fwd_launch(const PackShape& p, int n_tiles, int tile_rows, bool records) {
  const bool even = p.g() % 2 == 0;
  if (!even && tile_rows == 128) return {1, 1, direct_items((int64_t)n_tiles * p.Hq, 2 * kNumCU, records), false};
  const int64_t n_items = (int64_t)n_tiles * (even ? p.Hq / 2 : p.Hq);
  const FwdWay way = fwd_way(p, n_items, records);
  if (way == kHalves || (way == kSingles && even)) return {1, 1, true, way == kHalves};
  return {even ? 2 : 1, even ? 1 : 2, way != kQueues, false};
}

// Items of the backward's two kernels: key tiles (n_tiles) for n_split parts of each kv head's query heads, and query
// tiles (n_q_tiles) for every query head.
struct BwdItems {
  PackShape pack;
  int n_tiles, n_q_tiles, n_split;
  int heads() const { return pack.g() / n_split; }  // query heads a dK/dV item loops over
  int64_t dkdv() const { return (int64_t)n_tiles * pack.Hkv * n_split; }
  int64_t dq() const { return (int64_t)n_q_tiles * pack.Hq; }
};

// Eight or four wavefronts a key tile (dK/dV kernel).  Eight pay per step and cost per item, so the line is the mean
// number of steps an item has: heads of the item x blocks of 64 rows from the tile to its sample's end.  Time of the
// backward, four / eight, T = 512 to 32768, samples of one size and mixed ones:
//   d = 128, one head an item    samples of 60: .81 to .97; 250: .90 to .96; 600: .95 to .99; 1000: .98 to 1.01;
//                                1200: 1.00 to 1.01; 1500: 1.00 to 1.02; 2500: 1.02 to 1.03
//            two                 60: .92; 150: .98; 290: 1.02; 580: 1.03; 1000: 1.03
//            three and more      25: 1.01 (four) and 1.11 (eight); 60: 1.00 and 1.10; 250: 1.08; 1000: 1.06
//   d = 64, one                  25: 1.01; 60: 1.00; 126: .94 to .99; 240: 1.00 to 1.07; 800: 1.03 to 1.08
//            nine and more, no more items than compute units, d = 64 and 128: samples of 30 to 90: 1.12 to 1.25
// One or two heads with no more items than compute units: the launch is as long as its longest item, so eight from 100
// tokens a sample on (.995 to 1.39; of 60: .96 to .99).  Only a call without query tiles comes there: with them such a pack
// has one launch for dK/dV and dQ, always of eight (see one_launch).
inline bool eight_waves(const BwdItems& p) {
  const double len = p.pack.mean_len();
  const int heads = p.heads(), d = p.pack.d_qk;
  if (heads >= 3) return true;
  if (p.dkdv() <= kNumCU) return len >= 100;
  const double steps = heads * (len / 128 + 1);
  return steps >= (d == 64 ? 2.5 : heads == 2 ? 6.5 : 10);
}
// dK/dV and dQ in one launch (bwd_both_kernel), and with their items interleaved?  `rounds`: dK/dV items to a compute
// unit; heads: query heads an item loops over; len: tokens a sample.  Time of the backward, two launches / one, T = 512 to
// 50000; samples of 60, 250, 800, 3000 (log-normal) and one sample of .4 or .5 of the pack among short ones:
//   one head     interleaved.  To 1 round 1.3 to 1.75; to 3: 1.1 to 1.8.  Dispatched dK/dV first .94 to 1.6.
//     d = 64     to 5.5: 1.01 to 1.36; 5.9 to 12.9, len >= 900: .97 to 1.06; len <= 320, to 19: 1.01 to 1.08
//     d = 128    to 6.5: 1.02 to 1.20; 8.5 to 12: .97 (a sample of .5 to .7, len 1400 to 3000) to 1.08
//                len 150 to 350, to 15: 1.02 to 1.12; 18 to 25: .99 to 1.04; shorter, to 8: 1.02 to 1.18; to 12.7: .95 to 1.01
//   more heads   dK/dV first.  To 1 round 1.16 to 1.9.  Interleaved, two heads: .84 to 1.5 (as many dQ items as dK/dV, so
//                every second group of a die, and these go to the same of its shader engines); from four: .90 to 1.1
//     two        to 4: 1.03 to 1.63; 4.2: .99 to 1.04; len <= 320, to 5: 1.05 to 1.08
//     to five    to 4: 1.01 to 1.38 (d = 64, 3.1: .99, so to 2.9 there); 4.2 to 5.3: .98 to 1.02; len <= 100, to 12:
//                1.01 to 1.13
//     to eight   to 2.7: 1.00 to 1.29; 3.1 to 3.6: .97 to 1.03; len <= 100, to 12: 1.00 to 1.07.  Not measured beyond.
enum Launches { kTwo, kOne, kOneInterleaved };
inline Launches one_launch(const BwdItems& p) {
  if (p.n_tiles <= 0 || p.n_q_tiles <= 0 || p.dq() > 49 * 512) return kTwo;  // measured to 49 rounds of dQ
  const int heads = p.heads(), d = p.pack.d_qk;
  const double rounds = (double)p.dkdv() / kNumCU, len = p.pack.mean_len();
  if (heads == 1) {
    const bool one = d == 64 ? rounds <= (len <= 320 ? 19 : 5.5) : rounds <= (len < 150 ? 8 : len <= 350 ? 15 : 6.5);
    return !one ? kTwo : p.pack.Hq > 1 ? kOneInterleaved : kOne;
  }
  if (heads == 2) return rounds <= 4 || (len <= 320 && rounds <= 5) ? kOne : kTwo;
  const double most = heads <= 5 ? (d == 64 ? 2.9 : 4) : 2.7;
  return heads <= 8 && (rounds <= most || (len <= 100 && rounds <= 12)) ? kOne : kTwo;
}
// The same at head size 192 (bwd_both4_kernel): two launches / one, T = 512 to 16384, 8, 16 and 128 heads and 12/4:  to 1
// round 1.2 to 1.7; to 3: 1.04 to 1.77; to 4: 1.02 to 1.2; 4.2 to 5: .99 to 1.13; 6 to 10: .96 to 1.1; more: .95 to 1.0.
// Items of several heads were not measured.
inline bool one_launch4(const BwdItems& p) {
  if (p.n_tiles <= 0 || p.n_q_tiles <= 0 || p.dq() > 49 * 512) return false;
  return p.heads() == 1 && (double)p.dkdv() / kNumCU <= 4;
}
// The launches: one for dK/dV and dQ or two; eight: the dK/dV kernel of eight wavefronts (in a launch of its own).
// separate: the caller asked for records or events of either kernel, so each has its own launch (and gives the same bits).
struct BwdLaunch {
  bool one, interleaved, eight;
};
inline BwdLaunch bwd_launch(const BwdItems& p, bool separate) {
  if (p.pack.d_qk == 192) return {one_launch4(p) && !separate, false, false};
  const Launches way = one_launch(p);
  return {way != kTwo && !separate, way == kOneInterleaved, way != kTwo || eight_waves(p)};
}

}  // namespace hbp
