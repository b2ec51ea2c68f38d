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
// 256-row tiles) to a compute unit; `len`: tokens a sample.  Forward, time with queues and pairs or 256-row tiles / this way,
// T = 512 to 60000, 4 to 64 heads, samples of 60 to 1500 tokens (log-normal) alone / with one of .4 of the pack / of .7:
//   even, d = 64, singles           to 7, T to 16384           1.08 to 2.03 / 1.13 to 1.67 / 1.03 to 1.54
//                                   2 to 12, longer packs      1.10 to 1.66 / 1.05 to 1.18 / 1.02 to 1.10
//   even, d >= 128, singles         to 2                       1.03 to 1.91 / 1.00 to 1.72 / 1.05 to 1.55
//                                   2 to 2.7, len > 100        1.00 to 1.34 /  .99 to 1.35 /  .93 to 1.25
//                     len to 100    2 to 8, T to 8192          1.20 to 1.48 / 1.06 to 1.32 / -
//                                   2 to 12, longer packs      1.10 to 1.30 /  .95 to 1.29 / -
//     kv heads dealt evenly, pairs  2 to 4.8, T to 8192        1.00 to 1.41 / 1.04 to 1.31 / 1.02 to 1.29
//                                   4.8 to 7, T to 8192        1.01 to 1.29 / 1.03 to 1.17 / 1.00 to 1.06
//                                   2 to 4.8, longer packs     1.00 to 1.20 /  .99 to 1.08 / 1.00 to 1.05
//                                   4.8 to 12, longer packs     .96 to 1.21 /  .98 to 1.06 /  .98 to 1.02
//       singles there against pairs, 2 to 4.8                   .93 to 1.08 /  .92 to 1.12 /  .95 to 1.04
//     else, pairs                   2 to 2.7, T to 8192        1.28 to 1.34 / 1.13         / -
//                                   2 to 4.8, longer packs      .99 to 1.28 /  .96 to 1.18 /  .97 to 1.10
//                                   4.8 to 12                   .94 to 1.20 /  .96 to 1.07 /  .97 to 1.03
//   odd, 256-row tiles              to 3.5, T to 16384         1.00 to 1.88 / 1.00 to 1.59 / 1.00 to 1.36
//                                   3.5 to 5.5, T to 16384     1.01 to 1.53 /  .99 to 1.51 / 1.01 to 1.35
//                                   2 to 5.5, longer packs      .97 to 1.43 /  .95 to 1.20 /  .97 to 1.29
//                                   5.5 to 12                   .95 to 1.42 /  .95 to 1.42 /  .97 to 1.26
//   odd, kHalves: a workgroup of four wavefronts takes half of a 256-row tile: the longest item's chain of key tiles runs
//   without a second wavefront on its SIMD.  Against the better of 256-row tiles with queues and without:
//     d = 64          to 4.2                                    .99 to 1.45 / 1.02 to 1.27 /  .97 to 1.27
//                     4.2 to 7.5, len to 320                   1.34 to 1.53 / 1.04 to 1.24 /  .99 to 1.09
//                     beyond, to 12                            1.09 to 1.62 / 1.02 to 1.18 / 1.02 to 1.08
//     d = 128         to .75                                   1.03 to 1.22 /  .98 to 1.20 / 1.07 to 1.17
//                     .75 to 9, len to 350                     1.00 to 1.31 /  .98 to 1.22 /  .95 to 1.19
//                     .75 to 9, len > 350                       .91 to 1.20 /  .88 to 1.15 /  .92 to 1.15
//                     9 to 12, len to 350                      1.12 to 1.32 /  .97 to 1.13 /  .95 to  .98
//     d = 192         to 2.3                                    .93 to 1.21 /  .98 to 1.17 / 1.00 to 1.17
//                     2.3 to 6, len to 350                     1.02 to 1.27 /  .98 to 1.14 /  .96 to 1.09
//                     2.3 to 6, len > 350                       .93 to 1.10 /  .93 to 1.08 /  .96 to 1.05
//                     6 to 12, len to 350                      1.04 to 1.27 /  .96 to 1.07 /  .96 to  .99
//     len to 100      to 1.05                                  1.08 to 1.20 / 1.04 to 1.25 / -
//                     more, T to 16384                          .92 to 1.69 / 1.02 to 1.27 / -
//                     more, longer packs                       1.38 to 1.75 /  .99 to 1.25 / -
// The lines were drawn with an item's rows read a row a lane and two of a die's heads at a time without queues, where a way lost
// just behind its line.  The table is of the kernels as they are: no way loses within its lines but as shown, and several gain
// beyond them too; the lines have stayed.  The host knows the samples' mean length alone, so a line has to hold for packs with
// a very long sample beside short ones as well.
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
// backward in two launches, four / eight, T = 512 to 60000, more items than compute units, len tokens a sample (log-normal)
// alone / with a sample of .4 of the pack / of .7:
//                          len to 100                        200 to 400                        above 800
//   d = 64, one head        .98 to 1.07 / 1.05 to 1.11 / -    1.03 to 1.10 / 1.06 / 1.05        1.07 to 1.12 / 1.06 / 1.05
//           two            1.02 to 1.07 / 1.08 / -            1.10 to 1.13 / 1.08 / 1.06        1.11 / 1.07 / 1.06
//           four           1.12 to 1.16 / 1.09 / -            1.14 to 1.18 / 1.07 / 1.07        1.09 / 1.07 / 1.06
//   d = 128, one            .93 to 1.02 /  .99 to 1.07 / -     .96 to 1.07 / 1.00 / 1.02        1.01 to 1.06 / 1.00 / 1.02
//            two           1.03 to 1.10 / 1.03 / -            1.05 to 1.08 / 1.04 / 1.04        1.05 / 1.04 / 1.03
//            four, eight   1.10 to 1.19 / 1.04 / -            1.08 to 1.16 / 1.05 / 1.04        1.05 / 1.04 / 1.04
// (single figures: the least.)  In between, one head of 128: 100 to 200: .94 to 1.06 / .99 / 1.01; 400 to 800: .99 to 1.08 / 1.01
// / 1.01.  The lines were drawn with K and V read a row a lane, which cost eight wavefronts more; they have stayed.
// One or two heads with no more items than compute units: the launch is as long as its longest item, so eight from 100
// tokens a sample on.  Only a call without query tiles comes there: with them such a pack has one launch for dK/dV and dQ,
// always of eight (see one_launch).
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
// 60000, samples of 60 to 1500 tokens (log-normal) alone / with one of .4 of the pack / of .7; beyond a line, from there on:
//   one head     interleaved (dK/dV first, measured before an item's rows went through LDS: .94 to 1.6)
//     to 3       d = 64: 1.25 to 1.76 / 1.21 to 1.87 / 1.21 to 1.77; d = 128: 1.14 to 1.62 / 1.16 to 1.73 / 1.15 to 1.53
//     d = 64     3 to 5.5: 1.08 to 1.83 / 1.10 to 1.83 / 1.00 to 1.45; len to 320, to 19: 1.05 to 1.22 / .99 to 1.37 / .94 to 1.12
//                beyond 5.5, len > 320: .95 to 1.17 / .92 to 1.18 / .91 to 1.02
//     d = 128    3 to 6.5: 1.02 to 1.35 / 1.01 to 1.64 / .97 to 1.27; len 150 to 320, to 15: 1.01 to 1.15 / .98 to 1.20 /
//                .95 to 1.15; len to 150, 6.5 to 8.5: 1.08 to 1.19 / 1.16 to 1.20 / -; to 19: .97 to 1.14 / .99 to 1.19 / -
//                beyond 6.5, len > 320: .95 to 1.13 / .93 to 1.15 / .92 to 1.12
//   more heads   dK/dV first.  Interleaved, measured before, two heads: .84 to 1.5 (as many dQ items as dK/dV, so
//                every second group of a die, and these go to the same of its shader engines); from four: .90 to 1.1
//     two        to 4: 1.02 to 1.79 / 1.00 to 1.71 / 1.01 to 1.62; 4 to 5.5, len to 320: 1.07 to 1.26 / 1.02 to 1.37 / 1.02
//                to 1.04; longer: 1.01 to 1.05 / .95 to 1.09 / .97 to 1.05
//     four       to 2.9: 1.04 to 1.78 / 1.03 to 1.45 / 1.01 to 1.39; 3 to 4, d = 64: .99 to 1.18 / .99 to 1.42 / .98 to 1.08;
//                d = 128: 1.00 to 1.14 / .98 to 1.35 / .99 to 1.07; 4 to 5.5: .99 to 1.15 / .98 to 1.19 / .98 to 1.03; len to 150,
//                to 12: 1.01 to 1.13 / .99 to 1.13 / -
//     eight      to 2.7: 1.03 to 1.55 / 1.01 to 1.31 / .99 to 1.21; 3 to 4: .98 to 1.17 / .99 to 1.30 / .98 to 1.06; len to 150, to
//                12: 1.00 to 1.07 / .96 to 1.17 / -.  Not measured beyond eight.
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
// The same at head size 192 (bwd_both4_kernel), 16 heads: to 1 round 1.45 to 1.61; to 3: 1.07 to 1.75; to 4: 1.01 to 1.38; 4 to
// 5.5: .99 to 1.27; to 8.5: .99 to 1.17; to 12: .99 to 1.09; more: .98 to 1.06.  Items of several heads were not measured.
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
