// Launch shape of the packed cross-entropy: plain host functions, without HIP, so that a test without a GPU can ask them.
#pragma once
#include <stdint.h>

namespace hbp {

// Packs of up to kCePlanRows rows are planned in the main kernel, in LDS: one bit a row, a running count a word of 64 rows,
// and the bounds of up to kCePlanCu samples.
constexpr int kCePlanRows = 1 << 17;
constexpr int kCePlanCu = 1024;
constexpr int ce_plan_words(int T) { return (T + 63) / 64; }
constexpr int ce_plan_lds(int T, int n_samples) {
  return (ce_plan_words(T) + 1) * (int)(sizeof(uint64_t) + sizeof(int32_t)) + (n_samples <= kCePlanCu ? (n_samples + 1) * (int)sizeof(int32_t) : 0);
}
constexpr int kCeRowBatch = 256;  // rows whose scalars are staged in LDS at a time

// Whether rows are dealt in turn to the workgroups (see ce_main_kernel, with what was measured).
constexpr bool ce_dealt(int nt, int nch, bool hold, bool with_grad) { return with_grad && hold && nch * nt * 8 > 10240; }

// The most LDS that the main kernel's own arrays take: statistics of the wavefronts, two sets, and the counts of the
// planning; the rows' scalars; its range of rows.
constexpr int ce_own_lds(int nt, bool dealt) { return 5 * 4 * (nt / 64) + (dealt ? 5 : 3) * 4 * kCeRowBatch + 16; }

// The most workgroups a compute unit gets, if the registers allow for more: with more of them each has fewer rows, and
// they store into more rows at a time.  With the gradient, time with this many / with one fewer, T = 1000, 2500, 8192, all
// rows with a loss; 30 % without:
//   256 threads, V = 10248    .99, 1.02, 1.00; 1.00, 1.01, 1.01       512, V = 24576    .98,  .96, 1.00; 1.00, 1.02, 1.02
//                    12288   1.00,  .99, 1.00; 1.00, 1.03, 1.01                28672   1.00,  .98, 1.01; 1.04, 1.03, 1.02
//                    16384   1.00,  .99, 1.01; 1.00, 1.02, 1.01                32000    .84,  .88,  .91;  .82,  .92,  .95
//                                                                              45056    .88,  .90,  .95;  .84,  .97, 1.00
// The registers allow for one more at V = 16392 to 20480 and 32000 alone.  With this many / with one more:
//   512 threads, V = 16392    .95,  .88,  .96;  .93,  .93,  .95; 70 % without:  .94, 1.11,  .94
//                    20480    .98,  .86,  .94;  .96,  .92,  .96;                .92, 1.11,  .97
//                    32000   1.00, 1.00,  .98;  .94,  .97,  .98
// (with one more, rows of 16392 to 20480 were up to 6 % slower than cut by cost; with this many they are not.)
// Without it a workgroup has a row under way whatever its work is, so fewer are enough.  With 1 / 2 / 4 of 256 threads,
// V = 4096: 9.9 / 9.7 / 8.9, 16.0 / 13.4 / 11.8 and 37 / 28 / 23; 8000: 10.6 / 10.5 / 9.8, 17 / 15 / 14, 41 / 32 / 29 (8:
// 13.3 and 14.7 at T = 2500); with 1 / 2 of 512, V = 32000: 16.0 / 18.1, 26.6 / 29.3, 68 / 70; 65536: 24.6 / 29.7, 43.5 /
// 49.0, 130 / 129.
// A row that is streamed (hold false) has nothing under way over its reduction: two workgroups a unit, with the gradient
// and without.  Without it, one / two of 1024 threads, 30 % of the rows without a loss: V = 163848: T = 600: 30 / 28, 2500:
// 141 / 115, 8192: 403 / 333; 262144: T = 600: 49 / 42, 4096: 324 / 268; 400000: T = 2500: 313 / 258.  One is faster where
// the rows with a loss then go one to a unit (257 to 360 rows: T = 300: 19 / 26, 25 / 36, 33 / 50) or evenly two (T = 600,
// all with a loss, V = 202048: 48 / 54); the host does not know how many have one, and with one in every row T = 300 takes
// 30 / 26, 42 / 35, 58 / 48.
constexpr int ce_most_per_cu(int nt, int nch, bool hold, bool with_grad) {
  if (!hold) return 2;
  if (!with_grad) return nt == 256 ? 4 : 1;
  if (nt == 256) return nch <= 5 ? 8 : nch <= 7 ? 7 : 6;
  if (nt == 512) return nch <= 7 ? 3 : 2;
  return 2;
}
// Workgroups a compute unit holds at once; the main kernel's grid is that times the compute units.  One more would have
// its rows to itself, after the others: with the kernel's own arrays taken as 4 KiB and no pieces, a round of 256 workgroups
// on its own, us, that -> what fits: T = 98000, V = 10248: 856 -> 804; 100000, 14336: 1055 -> 1030; 120000, 16384: 1443 -> 1388.
constexpr int ce_per_cu(int by_registers, int nt, int nch, bool hold, bool with_grad, int plan_lds) {
  constexpr int kLds = 160 * 1024, kPiece = 1280;  // of a compute unit; the unit it is handed out in
  const int own = ce_own_lds(nt, ce_dealt(nt, nch, hold, with_grad));
  const int by_lds = kLds / ((plan_lds + own + kPiece - 1) / kPiece * kPiece);
  const int most = ce_most_per_cu(nt, nch, hold, with_grad);
  const int n = by_registers < most ? by_registers : most;
  return n < by_lds ? n : by_lds;
}

}  // namespace hbp
