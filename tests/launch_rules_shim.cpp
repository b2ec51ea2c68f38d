// The rules that choose a call's kernels and launches, for tests without a GPU.
#include "attn_rules.hpp"
#include "loss_rules.hpp"

// out: heads or pairs a workgroup (1, 2), 128-row halves a tile (1, 2), without queues?, halves of 256-row tiles?
extern "C" void fwd_route(int d_qk, int T, int n_samples, int Hq, int Hkv, int n_tiles, int tile_rows, int records, int* out) {
  const hbp::FwdLaunch l = hbp::fwd_launch(hbp::PackShape{d_qk, T, n_samples, Hq, Hkv}, n_tiles, tile_rows, records != 0);
  out[0] = l.hp; out[1] = l.tp; out[2] = l.direct; out[3] = l.halves;
}
// out: one launch?, interleaved?, eight wavefronts a key tile?, query heads a dK/dV item loops over, dK/dV and dQ items
extern "C" void bwd_route(int d_qk, int T, int n_samples, int Hq, int Hkv, int n_tiles, int n_q_tiles, int separate, int* out) {
  const hbp::BwdItems i{hbp::PackShape{d_qk, T, n_samples, Hq, Hkv}, n_tiles, n_q_tiles, hbp::heads_split(Hkv, Hq / Hkv)};
  const hbp::BwdLaunch l = hbp::bwd_launch(i, separate != 0);
  out[0] = l.one; out[1] = l.interleaved; out[2] = l.eight; out[3] = i.heads(); out[4] = (int)i.dkdv(); out[5] = (int)i.dq();
}
extern "C" int ce_per_cu(int threads, int chunks, int hold, int with_grad) {
  return hbp::ce_most_per_cu(threads, chunks, hold != 0, with_grad != 0);
}
// workgroups a compute unit of the cross-entropy's main kernel, as far as the registers allow for that many
extern "C" int ce_launched_per_cu(int threads, int chunks, int hold, int with_grad, int T, int n_samples) {
  return hbp::ce_per_cu(1 << 20, threads, chunks, hold != 0, with_grad != 0, T > hbp::kCePlanRows ? 0 : hbp::ce_plan_lds(T, n_samples));
}
extern "C" int ce_plan_lds(int T, int n_samples) { return hbp::ce_plan_lds(T, n_samples); }
// the most LDS that the main kernel's own arrays take
extern "C" int ce_own_lds(int threads, int chunks, int hold, int with_grad) {
  return hbp::ce_own_lds(threads, hbp::ce_dealt(threads, chunks, hold != 0, with_grad != 0));
}
