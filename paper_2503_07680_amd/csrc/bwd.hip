// Backward kernels: dQ, dK, dV of causal attention inside each sample of a packed buffer, gfx950.
//
// (1) prepass   D[h,r] = sum_x dO[r,h,x] O[r,h,x]; resets the scheduler counters of (2) and (3).
// (2) dq        query-tile major, same skeleton as the forward: work item = (query tile of <=128
//               rows, query head); K and V tiles of 64 keys stream through LDS; per 32-key block
//                   S^T  = K Q^T,  dP^T = V dO^T          (one query per lane column)
//                   dS^T = exp2(S^T c - LSE log2e) (dP^T - D)      (the dP^T accumulator starts at -D)
//                   dQ^T += K^T dS^T                      (K^T by transposing LDS reads)
// (3) dkdv      key-tile major: work item = (key tile of <=128 keys, kv head); each wavefront keeps
//               the K and V fragments of its 32 keys and the dK^T / dV^T accumulators in registers
//               while Q and dO blocks of 64 rows stream through LDS, for every query head of the
//               group (the GQA reduction happens in the accumulators):
//                   S  = Q K^T,  dP = dO V^T               (one key per lane column)
//                   P  = exp2(S c - LSE log2e),  dS = P (dP - D)
//                   dV^T += dO^T P,  dK^T += Q^T dS        (transposing LDS reads of dO and Q)
// No atomics: dQ has its own pass (S and dP are recomputed there), so every output is written
// once and the results are bit-stable from run to run.
#include <type_traits>

#include "common.hpp"

namespace hbp {

constexpr float kLog2e = 1.4426950408889634f;

// A kernel's first argument.  AGAIN: opaque to the optimiser, so that its members are read again here and not held in scalar
// registers over an item's loops, where spilled ones came back.
typedef const __attribute__((address_space(4))) BwdParams BwdArgs;
template <bool AGAIN>
__device__ __forceinline__ BwdArgs* bwd_args() {
  BwdArgs* a = (BwdArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  if (AGAIN) asm volatile("" : "+s"(a));
  return a;
}

struct ProfAcc {
  uint32_t n_done = 0;
  uint64_t t_first = 0, t_last = 0, t_busy = 0, t0 = 0;
};
__device__ __forceinline__ void prof_begin(ProfAcc& a, bool profiled, int tid) {
  if (profiled && tid == 0) {
    a.t0 = wall_clock64();
    if (a.n_done == 0) a.t_first = a.t0;
  }
}
__device__ __forceinline__ void prof_end(ProfAcc& a, bool profiled, int tid) {
  if (profiled && tid == 0) {
    const uint64_t t1 = wall_clock64();
    a.t_busy += t1 - a.t0;
    a.t_last = t1;
    ++a.n_done;
  }
}
__device__ __forceinline__ void prof_write(const ProfAcc& a, bool profiled, hbp_profile_rec* prof, int tid) {
  if (profiled && tid == 0) {
    hbp_profile_rec r;
    r.hw_id = hw_id_reg();
    r.xcc_id = xcc_id_reg();
    r.n_items = a.n_done;
    r.reserved = 0;
    r.first_tick = a.t_first;
    r.last_tick = a.t_last;
    r.busy_ticks = a.t_busy;
    prof[blockIdx.x] = r;
  }
}

// ------------------------------------------------------------------------------------- dQ
// Two workgroups per compute unit where the kernel fits 256 registers (d_qk <= 128): the second
// wavefront on each SIMD fills the issue slots the first one leaves open.
//
// HALVES = 2 (see bwd_both_kernel): the workgroup has eight wavefronts, four for each of two neighbouring query heads of
// the same tile, and takes the launch's item `block` alone.  SHARED: both heads read the same kv head and work off the
// same tiles in LDS (half the copies); otherwise each half has its own.
//
// Where a wavefront's rows of Q and dO go through LDS (RowStage): in the second K and V buffers, which take their first tile
// once every wavefront has read its rows, and behind the tiles; kBoth: beside each other, else one after the other.
template <int DQK, int DV, int HALVES, bool SHARED>
struct DqLds {
  static constexpr int NW = 4 * HALVES, K_TILE = 64 * DQK * 2, V_TILE = 64 * DV * 2, SETS = SHARED ? 1 : HALVES;
  static constexpr int TILES = SETS * 2 * (K_TILE + V_TILE), MOST = 160 * 1024 / (HALVES == 1 && DQK <= 128 ? 2 : 1);
  static constexpr bool kInTiles = DQK == DV;  // else all of them behind the tiles
  static constexpr int UNIT = RowStage<DQK>::BYTES, UNIT_V = RowStage<DV>::BYTES;
  static constexpr int IN_K = kInTiles ? K_TILE / UNIT : 0, IN_SET = 2 * IN_K, IN_TILES = SETS * IN_SET;
  static constexpr bool kBoth = kInTiles ? TILES + (2 * NW - IN_TILES) * UNIT <= MOST : true;
  static constexpr int UNITS = kBoth ? 2 * NW : NW;
  static constexpr int BYTES = kInTiles ? TILES + (UNITS > IN_TILES ? UNITS - IN_TILES : 0) * UNIT : TILES + NW * (UNIT + UNIT_V);
  static_assert(BYTES <= MOST && NW * UNIT <= TILES, "the compute unit's LDS; dQ's rows fit where the tiles were");
  // lds0: the workgroup's
  static __device__ __forceinline__ uint32_t unit(uint32_t lds0, int u) {
    if (u >= IN_TILES) return lds0 + TILES + (u - IN_TILES) * UNIT;
    const int set = u / (IN_SET ? IN_SET : 1), i = u - set * IN_SET;
    return lds0 + set * 2 * (K_TILE + V_TILE) + (i < IN_K ? K_TILE + i * UNIT : 2 * K_TILE + V_TILE + (i - IN_K) * UNIT);
  }
  static __device__ __forceinline__ uint32_t q_at(uint32_t lds0, int wave) {
    return kInTiles ? unit(lds0, wave) : lds0 + TILES + wave * (UNIT + UNIT_V);
  }
  static __device__ __forceinline__ uint32_t do_at(uint32_t lds0, int wave) {
    return kInTiles ? unit(lds0, kBoth ? NW + wave : wave) : lds0 + TILES + wave * (UNIT + UNIT_V) + UNIT;
  }
};

template <int DQK, int DV, int HALVES = 1, bool SHARED = false, bool DIRECT = HALVES == 2>
__device__ __forceinline__ void dq_items(int block) {
  using Lds = DqLds<DQK, DV, HALVES, SHARED>;
  constexpr int BM = 128, BN = 64;
  constexpr int KRB = DQK * 2, VRB = DV * 2;
  constexpr int K_TILE = BN * KRB, V_TILE = BN * VRB;
  constexpr int NC = DQK / 16, NCV = DV / 16, NDB = DQK / 32;
  constexpr int PD = DQK == 128 ? 3 : 4;  // read-ahead depth: at d = 128 the kernel is two registers short of its 256 with 4
  // Scores in the vector file (asm MFMA): needs a kernel that compiles without spills (checked at build
  // time); the builtin form stays as the fallback.
  constexpr bool kVgprScores = true;

  extern __shared__ __attribute__((aligned(1024))) char smem_all[];
  const int tid = threadIdx.x;
  const int wave_in_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = HALVES == 1 ? 0 : wave_in_wg >> 2;
  const int wave = (DQK > 64 ? mirrored(wave_in_wg) : wave_in_wg) & 3;  // its rows
  const int lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  // a half's [K buf0][K buf1][V buf0][V buf1]
  char* const smem = smem_all + (SHARED ? 0 : half * (2 * K_TILE + 2 * V_TILE));
  char* const k_lds = smem;
  char* const v_lds = smem + 2 * K_TILE;

  // Absolute LDS addresses of this lane's fragments: workgroup base and current buffer included
  // (toggled once per tile), so a read needs no address arithmetic.
  const uint32_t lds0 = lds_address(smem);
  // With equal row sizes (d_qk = d_v) a lane's V fragments sit exactly two K tiles behind its K fragments
  // (both buffers toggle together), so one set of addresses serves both.
  constexpr bool kSameRows = DQK == DV;
  uint32_t koff[NC], vnoff[kSameRows ? 1 : NCV], ktoff[2][NDB];
#pragma unroll
  for (int c = 0; c < NC; ++c) koff[c] = lds0 + l32 * KRB + swz<DQK>(2 * c + hh, l32) * 16;
  if (!kSameRows) {
#pragma unroll
    for (int c = 0; c < NCV; ++c) vnoff[c] = lds0 + 2 * K_TILE + l32 * VRB + swz<DV>(2 * c + hh, l32) * 16;
  }
  {
    const int G = lane >> 4, s = lane & 15;
    const int k8 = 4 * hh + (s >> 2);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int c = 4 * db + 2 * (G & 1) + ((s & 3) >> 1);
        ktoff[r][db] = lds0 + (8 * r + k8) * KRB + swz<DQK>(c, 8 * r + k8) * 16 + (s & 1) * 8;
      }
  }

  constexpr int NW = SHARED ? 8 : 4;  // wavefronts that copy a tile
  const int cwave = SHARED ? wave_in_wg : wave;
  TileLoader<DQK, BN, NW> k_loader;
  TileLoader<DV, BN, NW> v_loader;  // same lane pattern as k_loader when the row sizes agree: then only that one is kept
  k_loader.init(cwave, lane);
  if (!kSameRows) v_loader.init(cwave, lane);
  const uint32_t k_stride_b = (uint32_t)bwd_args<false>()->k_st * 2, v_stride_b = (uint32_t)bwd_args<false>()->v_st * 2;

  const bool profiled = !DIRECT && bwd_args<false>()->prof_dq;  // items of their own workgroup have no records
  ProfAcc pa;
  int q_cur = xcc_id_reg() & (kNumXcd - 1), q_tried = 0;
  for (;;) {
    const BwdArgs& p = *bwd_args<!DIRECT>();
    const WorkQueues wq{p.counter_dq, p.n_q_tiles, p.Hkv * p.n_split_dq, quotient(p.g / (SHARED ? 2 : 1), p.n_split_dq)};
    int tile_idx, h;
    if constexpr (!DIRECT) {
      if (!next_item(wq, (int*)smem, tid, q_cur, q_tried, tile_idx, h)) break;
    } else {
      const Taken tk = SHARED || HALVES == 1 ? direct_item_inline(wq.n_tiles, wq.Hkv, wq.per_kv, 0, 0, block)
                              : direct_item_inline(wq.n_tiles, (p.Hq + 1) / 2, 1, 0, 0, block);
      tile_idx = __builtin_amdgcn_readfirstlane(tk.tile_idx);
      h = HALVES * __builtin_amdgcn_readfirstlane(tk.head) + half;
    }
    prof_begin(pa, profiled, wave_in_wg);

    hbp_tile tl;
    int s0, s1;
    bool ok = load_tile(p.q_tiles, tile_idx, p.cu, p.n_samples, lane, tl, s0, s1);
    if (ok) {
      ok = s0 >= 0 && s1 <= p.T && s0 <= tl.row_begin && tl.row_begin < tl.row_end &&
           tl.row_end <= s1 && tl.row_end - tl.row_begin <= BM;
    }
    if (ok) {
      const int r0 = tl.row_begin, r1 = tl.row_end;
      const bool has_head = HALVES == 1 || SHARED || h < p.Hq;  // an odd number of heads: the last pair has one
      if (!has_head) h = p.Hq - 1;
      if (HALVES == 2) h = __builtin_amdgcn_readfirstlane(h);
      const int kh = quotient(h, p.g);
      const int qw0 = r0 - s0 + 32 * wave;
      const int my_row = r0 + 32 * wave + l32;
      const bool row_valid = has_head && my_row < r1;
      const bool wave_active = has_head && r0 + 32 * wave < r1;
      const int n_keys = r1 - s0;
      const int nkt = (n_keys + BN - 1) / BN;
      const uint16_t* kbase = p.k + (int64_t)s0 * p.k_st + (int64_t)kh * p.k_sh;
      const uint16_t* vbase = p.v + (int64_t)s0 * p.v_st + (int64_t)kh * p.v_sh;

      // copy `slot` of this wave's share of key tile kt (K first, then V)
      constexpr int NKCP = decltype(k_loader)::PER_WAVE, NVCP = decltype(v_loader)::PER_WAVE;
      auto issue_slot = [&](int kt, int slot) {
        const int k_off = kt * BN;
        const int valid = n_keys - k_off;
        if (slot < NKCP) {
          k_loader.issue_one(slot, kbase + (int64_t)k_off * p.k_st, k_stride_b, valid, k_lds + (kt & 1) * K_TILE, cwave);
        } else if constexpr (kSameRows) {
          k_loader.issue_one(slot - NKCP, vbase + (int64_t)k_off * p.v_st, v_stride_b, valid, v_lds + (kt & 1) * V_TILE, cwave);
        } else {
          v_loader.issue_one(slot - NKCP, vbase + (int64_t)k_off * p.v_st, v_stride_b, valid, v_lds + (kt & 1) * V_TILE, cwave);
        }
      };
      auto issue = [&](int kt) {
#pragma unroll
        for (int slot = 0; slot < NKCP + NVCP; ++slot) issue_slot(kt, slot);
      };
      Frag qf[NC], dof[NCV];
      float lse2 = INFINITY, Dv = 0.f;  // +inf: rows past the tile end get probability 0
      if (row_valid) {
        lse2 = p.lse2[(int64_t)h * p.T + my_row];
        Dv = p.D[(int64_t)h * p.T + my_row];
      }
      const uint32_t lds_all = lds_address(smem_all);
      const int first_row = r0 + 32 * wave;  // of this wave
      {
        const uint16_t* q_rows = p.q + (int64_t)first_row * p.q_st + (int64_t)h * p.q_sh;
        const uint16_t* do_rows = p.d_o + (int64_t)first_row * p.o_st + (int64_t)h * p.o_sh;
        const uint32_t q_at = Lds::q_at(lds_all, wave_in_wg), do_at = Lds::do_at(lds_all, wave_in_wg);
        const int rows = has_head ? r1 - first_row : 0;
        RowStage<DQK>::copy_in(q_rows, (uint32_t)p.q_st * 2, rows, q_at, lane);
        if (Lds::kBoth) RowStage<DV>::copy_in(do_rows, (uint32_t)p.o_st * 2, rows, do_at, lane);
        issue(0);
        wait_async_but<NKCP + NVCP>();
        RowStage<DQK>::fragments(q_at, lane, qf);
        if constexpr (!Lds::kBoth) {
          wait_lds_reads();
          RowStage<DV>::copy_in(do_rows, (uint32_t)p.o_st * 2, rows, do_at, lane);
          wait_async_loads();
        }
        RowStage<DV>::fragments(do_at, lane, dof);
        race_fence();
      }
      // the dP^T accumulator of every block starts at -D of the lane's query (one value per lane): the
      // subtraction in dS = P (dP - D) then comes out of the MFMAs
      f32x16 negD;
#pragma unroll
      for (int i = 0; i < 16; ++i) negD[i] = -Dv;
      asm volatile("" : "+v"(negD));
      f32x16 dqacc[NDB];
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dqacc[db][i] = 0.f;
      const int q_in = qw0 + l32;

      // One 32-key block: sd = (S^T, dP^T - D) products, sm = dS^T = exp2(c S^T - LSE2)(dP^T - D),
      // gr = dQ^T += K^T dS^T.  Interior tiles pipeline their two blocks inside the wave:
      //     sd(0) | sd(1) + sm(0) | gr(0) + sm(1) first half | gr(1) first half + sm(1) rest | gr(1) rest
      struct Blk {
        f32x16 s, dp;
        Frag dsf[2];
      };
      // buf: a compile-time tile buffer on top of where the lane's offsets point (the interior loop names
      // the second buffer this way, in the reads' immediate offsets, instead of moving the offsets per tile)
      auto sd_load = [&](int blk, int buf = 0) {
        return [&, blk, buf](int i) {
          const int ka = 32 * blk * KRB + buf * K_TILE, va = 32 * blk * VRB + buf * V_TILE;
          Frag a;
          if (i < NC) a.u = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(koff[i] + ka);
          else if (kSameRows) a.u = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(koff[i - NC] + (2 * K_TILE + va));
          else a.u = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(vnoff[i - NC] + va);
          return a;
        };
      };
      auto sd_mma = [&](Blk& x) {
        return [&](int i, const Frag& a) {
          if (kVgprScores) {
            if (i == 0) x.s = mfma32_vgpr_first(a.v, qf[0].v);
            else if (i < NC) mfma32_vgpr(x.s, a.v, qf[i].v);
            else if (i == NC) x.dp = mfma32_vgpr_from(a.v, dof[0].v, negD);  // starts at -D: ends as dP - D
            else mfma32_vgpr(x.dp, a.v, dof[i - NC].v);
          } else {
            if (i == 0 || i == NC) {
              f32x16 z;
#pragma unroll
              for (int e = 0; e < 16; ++e) z[e] = 0.f;
              if (i == 0) x.s = mfma32(a.v, qf[0].v, z);
              else x.dp = mfma32(a.v, dof[0].v, negD);
            } else if (i < NC) {
              x.s = mfma32(a.v, qf[i].v, x.s);
            } else {
              x.dp = mfma32(a.v, dof[i - NC].v, x.dp);
            }
          }
        };
      };
      auto gr_frag = [&](int blk, int j, int db, int buf = 0) {
        const uint32_t base = (32 * blk + 16 * j) * KRB + buf * K_TILE;
        Frag a;
        a.h[0] = lds_read_tr16_at(ktoff[0][db] + base);
        a.h[1] = lds_read_tr16_at(ktoff[1][db] + base);
        return a;
      };
      // slices 0..16 of a block: slice k issues exp for element k (k < 16) and finishes element
      // k-1 (k > 0); element e = 4b+v <-> key 32 blk + 8b + 4hh + v of the tile, query column q_in
      float e_cur = 0.f, ds_even = 0.f;
      auto sm_slice = [&](Blk& x, int kb, int k, auto masked) {
        const float e_prev = e_cur;
        if (k < 16) e_cur = __builtin_amdgcn_exp2f(__builtin_fmaf(x.s[k], p.scale_log2, -lse2));
        if (k > 0) {
          const int e = k - 1;
          float pr = e_prev;
          if (decltype(masked)::value) {
            if (kb + 8 * (e >> 2) + 4 * hh + (e & 3) > q_in) pr = 0.f;
          }
          const float ds = pr * x.dp[e];
          if (e & 1) x.dsf[e >> 3].w[(e & 7) >> 1] = pack_bf16(ds_even, ds);
          else ds_even = ds;
        }
      };

      int cur_buf = 0;
      auto point_offsets_at = [&](int buf) {
        const int dk = buf ? K_TILE : -K_TILE, dv = buf ? V_TILE : -V_TILE;
#pragma unroll
        for (int c = 0; c < NC; ++c) koff[c] += dk;
        if (!kSameRows) {
#pragma unroll
          for (int c = 0; c < NCV; ++c) vnoff[c] += dv;
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int db = 0; db < NDB; ++db) ktoff[r][db] += dk;
        cur_buf = buf;
      };
      // copies_now: the next tile's copies go out here in one go; an interior tile spreads them behind the MFMAs
      // of its first chain instead (a tile follows every interior tile)
      auto begin_tile = [&](int kt, bool point = true, bool copies_now = true) {
        race_fence();
        wait_async_loads();
        __syncthreads();
        if (copies_now && kt + 1 < nkt) issue(kt + 1);
        if (point && (kt & 1) != cur_buf) point_offsets_at(kt & 1);
      };

      const int n_interior = wave_active ? min(nkt, (qw0 + 1) / BN) : 0;
      // One interior tile.  BUF = kt & 1 as a compile-time constant: the lane's offsets stay on buffer 0
      // and the reads carry the buffer in their immediate offsets; BUF < 0: the offsets follow the buffers.
      auto interior_tile = [&](auto bufc, int kt) {
        constexpr int BUF = decltype(bufc)::value < 0 ? 0 : decltype(bufc)::value;
        begin_tile(kt, decltype(bufc)::value < 0, false);
        const int k_off = kt * BN;
        Blk x0, x1;
        LdsChain<NC + NCV, PD> c1;
        c1.prefill(sd_load(0, BUF));
        c1.template run_with<NKCP + NVCP>(sd_load(0, BUF), sd_mma(x0), [&](int slot) { issue_slot(kt + 1, slot); });
        c1.prefill(sd_load(1, BUF));
        if (kVgprScores) mfma_results_ready(x0.s, x0.dp);
        c1.template run_with<17>(sd_load(1, BUF), sd_mma(x1), [&](int k) { sm_slice(x0, k_off, k, std::false_type{}); });
        // gr(0) (2*NDB MFMAs) then gr(1) j=0 (NDB) then gr(1) j=1 (NDB), with sm(1) spread so that
        // dS chunk j of block 1 is complete before the MFMAs that read it
        constexpr int LG = 4 * NDB;
        auto g_load = [&](int i) {
          const int blk = i / (2 * NDB), j = (i / NDB) & 1, db = i % NDB;
          return gr_frag(blk, j, db, BUF);
        };
        LdsChain<LG, PD> c2;
        c2.prefill(g_load);
        if (kVgprScores) mfma_results_ready(x1.s, x1.dp);
#pragma unroll
        for (int i = 0; i < LG; ++i) {
          const int blk = i / (2 * NDB), j = (i / NDB) & 1, db = i % NDB;
          Blk& x = blk ? x1 : x0;
          dqacc[db] = mfma32(c2.ring[i % PD].v, x.dsf[j].v, dqacc[db]);
          if (i + PD < LG) c2.ring[i % PD] = g_load(i + PD);
          // sm(1): slices 0..8 behind gr(0) (chunk 0 of block 1 done), 9..16 behind gr(1) j=0
          constexpr int A = 2 * NDB, B = NDB;
          if (i < A) {
#pragma unroll
            for (int k = i * 9 / A; k < (i + 1) * 9 / A; ++k) sm_slice(x1, k_off + 32, k, std::false_type{});
          } else if (i < A + B) {
#pragma unroll
            for (int k = 9 + (i - A) * 8 / B; k < 9 + (i - A + 1) * 8 / B; ++k)
              sm_slice(x1, k_off + 32, k, std::false_type{});
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      int kt = 0;  // the offsets point at buffer 0 here
      for (; kt + 1 < n_interior; kt += 2) {
        interior_tile(std::integral_constant<int, 0>{}, kt);
        interior_tile(std::integral_constant<int, 1>{}, kt + 1);
      }
      for (; kt < n_interior; ++kt) interior_tile(std::integral_constant<int, -1>{}, kt);
      for (; kt < nkt; ++kt) {  // tiles that touch the diagonal: plain masked path, block by block
        begin_tile(kt);
        const int k_off = kt * BN;
        if (!wave_active || k_off > qw0 + 31) continue;
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          const int kb = k_off + 32 * blk;
          if (kb > qw0 + 31) continue;
          Blk x;
          LdsChain<NC + NCV, PD> c1;
          c1.prefill(sd_load(blk));
          c1.run(sd_load(blk), sd_mma(x));
          auto g_load = [&](int i) { return gr_frag(blk, i / NDB, i % NDB); };
          LdsChain<2 * NDB, PD> c2;
          c2.prefill(g_load);
          if (kVgprScores) mfma_results_ready(x.s, x.dp);
#pragma unroll
          for (int k = 0; k < 17; ++k) sm_slice(x, kb, k, std::true_type{});
          __builtin_amdgcn_sched_barrier(0);
          c2.run(g_load, [&](int i, const Frag& a) { dqacc[i % NDB] = mfma32(a.v, x.dsf[i / NDB].v, dqacc[i % NDB]); });
        }
      }
      if (cur_buf) point_offsets_at(0);

      __syncthreads();  // the tiles are no longer read
      race_fence();
      if (wave_active) {
        const uint32_t at = lds_all + wave_in_wg * Lds::UNIT;
        RowStage<DQK>::put(at, lane, dqacc, p.scale);
        RowStage<DQK>::copy_out(p.dq + (int64_t)first_row * p.q_st + (int64_t)h * p.q_sh, (uint32_t)p.q_st * 2, r1 - first_row, at, lane);
      }
    }
    prof_end(pa, profiled, wave_in_wg);
    if constexpr (DIRECT) break;
  }
  prof_write(pa, profiled, bwd_args<false>()->prof_dq, tid);
}
template <int DQK, int DV>
__global__ __launch_bounds__(kThreads, DQK <= 128 ? 2 : 1) void bwd_dq_kernel(const BwdParams) {
  dq_items<DQK, DV>(0);
}

// ----------------------------------------------------------------------------------- dK, dV
// Where a wavefront's rows of K and V go through LDS (RowStage): behind the tiles, the last wavefront's rows of V where the
// second Q buffer is, or at head size 192 it would not fit the compute unit's LDS.  (An item of one step, whose idle step
// multiplies what is there by zero, has no rows for that wavefront: its copies write zeros.)
template <int DQK, int DV>
struct DkdvLds {
  static constexpr int TILES = 2 * 64 * (DQK * 2 + DV * 2) + 4 * 64 * (int)sizeof(float);
  static constexpr int K = RowStage<DQK>::BYTES, V = RowStage<DV>::BYTES;
  static constexpr int bytes() { return TILES + 4 * K + 3 * V; }
  static_assert(bytes() <= 160 * 1024 && V <= 64 * DQK * 2 && DV <= DQK, "LDS of a compute unit");
  static __device__ __forceinline__ uint32_t k_at(uint32_t lds0, int wave) { return lds0 + TILES + wave * K; }
  static __device__ __forceinline__ uint32_t v_at(uint32_t lds0, int wave) {
    return wave < 3 ? lds0 + TILES + 4 * K + wave * V : lds0 + 64 * DQK * 2;
  }
};

// DIRECT: the launch's item `block` and no other (see bwd_both4_kernel).  n_resident: workgroups under way at a time.
template <int DQK, int DV, bool DIRECT = false>
__device__ __forceinline__ void dkdv_items(int block, int n_resident) {
  constexpr int BN = 128, BQ = 64;
  constexpr int QRB = DQK * 2, ORB = DV * 2;
  constexpr int Q_TILE = BQ * QRB, O_TILE = BQ * ORB;
  constexpr int NC = DQK / 16, NCV = DV / 16, NDB = DQK / 32, NEB = DV / 32;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // [Q buf0][Q buf1][dO buf0][dO buf1][lse buf0|buf1][D buf0|buf1]
  char* const q_lds = smem;
  char* const o_lds = smem + 2 * Q_TILE;
  float* const lse_lds = (float*)(smem + 2 * Q_TILE + 2 * O_TILE);
  float* const d_lds = lse_lds + 2 * BQ;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hh = lane >> 5;

  // Absolute LDS addresses of this lane's fragments in buffer 0 (workgroup base included): a read
  // needs no address arithmetic, the buffer and the sub-block go into its immediate offset.
  const uint32_t lds0 = lds_address(smem);
  uint32_t qoff[NC], dooff[NCV], qtoff[2][NDB], dotoff[2][NEB];
#pragma unroll
  for (int c = 0; c < NC; ++c) qoff[c] = lds0 + l32 * QRB + swz<DQK>(2 * c + hh, l32) * 16;
#pragma unroll
  for (int c = 0; c < NCV; ++c) dooff[c] = lds0 + 2 * Q_TILE + l32 * ORB + swz<DV>(2 * c + hh, l32) * 16;
  {
    const int G = lane >> 4, s = lane & 15;
    const int k8 = 4 * hh + (s >> 2);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int c = 4 * db + 2 * (G & 1) + ((s & 3) >> 1);
        qtoff[r][db] = lds0 + (8 * r + k8) * QRB + swz<DQK>(c, 8 * r + k8) * 16 + (s & 1) * 8;
      }
#pragma unroll
      for (int eb = 0; eb < NEB; ++eb) {
        const int c = 4 * eb + 2 * (G & 1) + ((s & 3) >> 1);
        dotoff[r][eb] = lds0 + 2 * Q_TILE + (8 * r + k8) * ORB + swz<DV>(c, 8 * r + k8) * 16 + (s & 1) * 8;
      }
    }
  }
  // LDS addresses of this lane's LSE2 / D rows inside the current buffer
  uint32_t lseoff = lds0 + 2 * Q_TILE + 2 * O_TILE + 16 * hh;
  uint32_t dvoff = lseoff + 2 * BQ * 4;

  const uint32_t q_stride_b = (uint32_t)bwd_args<false>()->q_st * 2, o_stride_b = (uint32_t)bwd_args<false>()->o_st * 2;
  FullTileLoader<DQK, BQ> q_loader;
  FullTileLoader<DV, BQ> o_loader;
  q_loader.init(wave, lane, q_stride_b);
  o_loader.init(wave, lane, o_stride_b);

  // Both tile buffers start out as zeros: an idle step (see the step loop) multiplies whatever the
  // second buffer holds by zero operands, and that must not be the NaN patterns of unwritten LDS.
  for (int i = tid * 16; i < 2 * Q_TILE + 2 * O_TILE + 4 * BQ * (int)sizeof(float); i += kThreads * 16)
    *(u32x4*)(smem + i) = u32x4{0, 0, 0, 0};
  __syncthreads();

  using Lds = DkdvLds<DQK, DV>;
  const bool profiled = !DIRECT && bwd_args<false>()->prof;
  ProfAcc pa;
  // Work item = (key tile, kv head, part of its query heads): with n_split > 1 the g heads of a kv head
  // are cut into n_split runs of g_item heads, each an item of its own.
  int q_cur = xcc_id_reg() & (kNumXcd - 1), q_tried = 0;
  for (;;) {
    const BwdArgs& p = *bwd_args<!DIRECT>();
    const WorkQueues wq{p.counter, p.n_tiles, p.Hkv * p.n_split, 1};
    const int g_item = quotient(p.g, p.n_split);
    int tile_idx, vh;
    if constexpr (DIRECT) {
      const Taken tk = direct_item_inline(wq.n_tiles, wq.Hkv, 1, 0, 0, block);
      tile_idx = __builtin_amdgcn_readfirstlane(tk.tile_idx);
      vh = __builtin_amdgcn_readfirstlane(tk.head);
    } else {
      if (!next_item(wq, (int*)smem, tid, q_cur, q_tried, tile_idx, vh)) break;
    }
    const int kh = quotient(vh, p.n_split), part = vh - kh * p.n_split;
    const int head0 = vh * g_item;  // first query head of the item
    prof_begin(pa, profiled, tid);

    hbp_tile tl;
    int s0, s1;
    bool ok = load_tile(p.tiles, tile_idx, p.cu, p.n_samples, lane, tl, s0, s1);
    if (ok) {
      ok = s0 >= 0 && s1 <= p.T && s0 <= tl.row_begin && tl.row_begin < tl.row_end &&
           tl.row_end <= s1 && tl.row_end - tl.row_begin <= BN;
    }
    if (ok) {
      const int s_len = s1 - s0;
      const int k0_in = tl.row_begin - s0;
      const int kw0_in = k0_in + 32 * wave;
      const int my_key = tl.row_begin + 32 * wave + l32;
      const bool key_valid = my_key < tl.row_end;
      const bool wave_active = tl.row_begin + 32 * wave < tl.row_end;
      const int key_in = kw0_in + l32;

      const int qb_start = (k0_in / BQ) * BQ;
      const int nqb = (s_len - qb_start + BQ - 1) / BQ;
      const int n_steps = nqb * g_item;

      // Step order: the query blocks from the LAST one of the sample down to the tile's own, and for each
      // block the g query heads of the group.  Every key tile of a sample needs a suffix of the same
      // blocks, so the workgroups of a die (they work on tiles of the same kv head) ask for the same
      // block at about the same time and it comes from that die's L2 once, not from HBM once per tile.
      // That only works while they walk in step: 32 workgroups two blocks apart put 8 MB between two
      // uses of a block, more than the L2 holds.  The w workgroups that share a kv head take the tiles
      // of a long sample w at a time, longest first.  Tiles 0..w-1 start together and end BN/BQ blocks
      // apart (each is that much shorter than the one before); their workgroups then take tiles
      // w..2w-1 one after the other, BN/BQ blocks apart.  Such a tile starts as many blocks below the top
      // as it starts late (where the first tile of its set is by then) and does the blocks it skipped at
      // the end; that set of w tiles ends together, the next one starts together, and so on in turns.  The
      // order is a function of the tile number alone, so the results do not depend on timing.
      // (With fewer than 8 workgroups per kv head there is little to share and the plain order is kept.)
      const int w_share = quotient(n_resident, min(p.Hkv * p.n_split, kNumXcd * kHeadGroup));  // heads in work at a time
      const int set = quotient(tl.tile, max(w_share, 1));
      int skip = w_share >= 8 && (set & 1) ? (tl.tile - set * w_share) * (BN / BQ) : 0;
      skip = max(0, min(skip, nqb - 1));
      const int first_blk = nqb - 1 - skip;
      // the blocks are taken in the order first_blk .. 0, then nqb-1 .. first_blk+1, g steps each
      // Copies are issued in step order; the source pointers of the next block to copy are carried
      // along instead of being recomputed from the step number.
      const int64_t first_row = (int64_t)s0 + qb_start + (int64_t)first_blk * BQ;
      const uint16_t* q_blk = p.q + first_row * p.q_st + (int64_t)head0 * p.q_sh;
      const uint16_t* o_blk = p.d_o + first_row * p.o_st + (int64_t)head0 * p.o_sh;
      const float* row_blk = (wave == 0 ? p.lse2 : p.D) + (int64_t)head0 * p.T + first_row;
      const uint16_t* q_src = q_blk;
      const uint16_t* o_src = o_blk;
      const float* row_src = row_blk;
      int blk_next = first_blk, head_next = 0;
      // The copies of a step's operands are issued one at a time (slot 0 .. N_COPY-1), so that they can sit
      // behind the MFMAs of the step before; taking the last slot moves the source on to the next step.
      // qb_in[buf]: first query row (in-sample) of the block whose copies went to buffer buf.
      constexpr int NQC = decltype(q_loader)::PER_WAVE, NOC = decltype(o_loader)::PER_WAVE;
      constexpr int N_COPY = NQC + NOC + 1;
      int qb_in[2] = {0, 0};
      // FULL: all BQ rows of the block exist (no clamping of the source rows, no vector arithmetic at all)
      auto issue_copy = [&](int slot, int buf, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int valid = FULL ? BQ : s_len - qb_start - blk_next * BQ;  // >= 1; < BQ only for the sample's last block
        if (slot < NQC) {
          if (FULL) q_loader.issue_full(slot, q_src, q_lds + buf * Q_TILE, wave);
          else q_loader.issue_one(slot, q_src, q_stride_b, valid, q_lds + buf * Q_TILE, wave, lane);
        } else if (slot < NQC + NOC) {
          if (FULL) o_loader.issue_full(slot - NQC, o_src, o_lds + buf * O_TILE, wave);
          else o_loader.issue_one(slot - NQC, o_src, o_stride_b, valid, o_lds + buf * O_TILE, wave, lane);
        } else {
          if (wave < 2) {
            // issued through the same untracked path as the tiles: the compiler must not see an LDS
            // write here, or it would drain every outstanding copy before the next LDS read
            const int row = lane < valid ? lane : valid - 1;
            const float* dst = (wave == 0 ? lse_lds : d_lds) + buf * BQ;
            async_copy4(row_src, (uint32_t)row * 4u, lds_address(dst));
          }
          qb_in[buf] = qb_start + blk_next * BQ;
          if (++head_next == g_item) {  // on to the block before; from the tile's own block to the sample's last
            head_next = 0;
            const int64_t jump = blk_next == 0 ? (int64_t)(nqb - 1) * BQ : -(int64_t)BQ;
            blk_next = blk_next == 0 ? nqb - 1 : blk_next - 1;
            q_blk += jump * p.q_st;
            o_blk += jump * p.o_st;
            row_blk += jump;
            q_src = q_blk;
            o_src = o_blk;
            row_src = row_blk;
          } else {
            q_src += p.q_sh;
            o_src += p.o_sh;
            row_src += p.T;
          }
        }
      };
      auto next_is_full = [&]() { return s_len - qb_start - blk_next * BQ >= BQ; };
      auto issue_next = [&](int buf) {  // all of a step's copies in one go
#pragma unroll
        for (int slot = 0; slot < N_COPY; ++slot) issue_copy(slot, buf, std::false_type{});
      };
      // register-resident B operands of this wave's 32 keys: lane column = key l32
      const uint32_t k_at = Lds::k_at(lds0, wave), v_at = Lds::v_at(lds0, wave);
      const int first_key = tl.row_begin + 32 * wave;  // of this wave
      RowStage<DQK>::copy_in(p.k + (int64_t)first_key * p.k_st + (int64_t)kh * p.k_sh, (uint32_t)p.k_st * 2, tl.row_end - first_key, k_at, lane);
      RowStage<DV>::copy_in(p.v + (int64_t)first_key * p.v_st + (int64_t)kh * p.v_sh, (uint32_t)p.v_st * 2, tl.row_end - first_key, v_at, lane);
      if (n_steps > 0) issue_next(0);
      wait_async_but<NQC + NOC>();  // a wave copies its share of the tiles and, the first two, of the rows' scalars too

      Frag knat[NC], vnat[NCV];
      {
        RowStage<DQK>::fragments(k_at, lane, knat);
        RowStage<DV>::fragments(v_at, lane, vnat);
        race_fence();
#pragma unroll
        for (int c = 0; c < NCV; ++c) vnat[c].u ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
      }
      f32x16 dkt[NDB], dvt[NEB];
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dkt[db][i] = 0.f;
#pragma unroll
      for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
        for (int i = 0; i < 16; ++i) dvt[eb][i] = 0.f;

      // One 32-query x 32-key sub-block: sd = (S, dP) products, sm = probabilities and dS,
      // gr = dV^T / dK^T updates.  Away from the diagonal two sub-blocks are software-pipelined
      // inside the wave so the vector arithmetic of one is spread, one element per MFMA, behind the
      // other's MFMAs (the matrix pipe leaves about half of each MFMA's issue time free):
      //     sd(A) | sd(B) + sm(A) | gr(A) + sm(B) | gr(B)
      // Blocks that touch the diagonal or the sample tail take the plain masked path.
      struct Sub {
        f32x16 s, dp;
        Frag pb[2], dsb[2];
      };
      constexpr int kPD = 3;  // LDS read-ahead depth (fragments)
      // active: a step of the item (not the idle one that makes the count even); has_next: another step
      // follows, whose operands this step copies into the other buffer.
      auto do_step = [&](auto buf_tag, bool active, bool has_next) {
        // the step's buffer is a compile-time constant: it goes into the immediate offset of every LDS
        // read (two copies of the step's code instead of 34 address updates per step)
        constexpr int BUF = decltype(buf_tag)::value;
        const int qb = qb_in[BUF];
        auto sd_load = [&](int sub) {
          return [&, sub](int i) {
            Frag a;
            if (i < NC) a.u = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(qoff[i] + 32 * sub * QRB + BUF * Q_TILE);
            else a.u = *(const __attribute__((address_space(3))) u32x4*)(uintptr_t)(dooff[i - NC] + 32 * sub * ORB + BUF * O_TILE);
            return a;
          };
        };
        // The asm form (scores produced in the vector file) needs a kernel that compiles without
        // register spills: spill copies next to an asm MFMA would bypass the compiler's hazard
        // handling.  Every instantiation does (a build-time test checks it); the builtin form stays
        // as the fallback should one stop doing so.
        constexpr bool kVgprScores = true;
        auto sd_mma = [&](Sub& x) {
          return [&](int i, const Frag& a) {
            if (kVgprScores) {
              if (i == 0) x.s = mfma32_vgpr_first(a.v, knat[0].v);
              else if (i < NC) mfma32_vgpr(x.s, a.v, knat[i].v);
              else if (i == NC) mfma32_vgpr(x.dp, a.v, vnat[0].v);
              else mfma32_vgpr(x.dp, a.v, vnat[i - NC].v);
            } else {
              if (i == 0 || i == NC) {
                f32x16 z;
#pragma unroll
                for (int e = 0; e < 16; ++e) z[e] = 0.f;
                if (i == 0) x.s = mfma32(a.v, knat[0].v, z);
                else x.dp = mfma32(a.v, vnat[0].v, z);
              } else if (i < NC) {
                x.s = mfma32(a.v, knat[i].v, x.s);
              } else {
                x.dp = mfma32(a.v, vnat[i - NC].v, x.dp);
              }
            }
          };
        };
        auto gr_load = [&](int sub) {
          return [&, sub](int i) {
            Frag a;
            if (i < 2 * NEB) {
              const int eb = i % NEB, j = i / NEB;
              const uint32_t base = (32 * sub + 16 * j) * ORB + BUF * O_TILE;
              a.h[0] = lds_read_tr16_at(dotoff[0][eb] + base);
              a.h[1] = lds_read_tr16_at(dotoff[1][eb] + base);
            } else {
              const int db = (i - 2 * NEB) % NDB, j = (i - 2 * NEB) / NDB;
              const uint32_t base = (32 * sub + 16 * j) * QRB + BUF * Q_TILE;
              a.h[0] = lds_read_tr16_at(qtoff[0][db] + base);
              a.h[1] = lds_read_tr16_at(qtoff[1][db] + base);
            }
            return a;
          };
        };
        auto gr_mma = [&](Sub& x) {
          return [&](int i, const Frag& a) {
            if (i < 2 * NEB) dvt[i % NEB] = mfma32(a.v, x.pb[i / NEB].v, dvt[i % NEB]);
            else dkt[(i - 2 * NEB) % NDB] = mfma32(a.v, x.dsb[(i - 2 * NEB) / NDB].v, dkt[(i - 2 * NEB) % NDB]);
          };
        };
        // element i = 4b+v of the accumulators <-> query q0 + 8b + 4hh + v, key column key_in.
        // The per-element arithmetic  pr = exp2(c*s - lse2);  ds = pr * (D - dP)  is issued in two
        // stages one slice apart (stage 1 of element i next to stage 2 of element i-1), so that no
        // vector instruction waits on the one just before it; LSE2 of the 4 query rows of group b is
        // read from LDS one group ahead (rows_prefetch(sub, 0) before the chain).  D - dP comes
        // straight out of the MFMAs: the accumulator starts as D (init_dp) and V is held negated, so
        // no subtraction is left for the vector unit; dS and dK carry the opposite sign until the
        // final scaling.
        f32x4 l4, l4n;
        float e_cur = 0.f;  // exp of element i (stage 1)
        float pr_even = 0.f, ds_even = 0.f;
        auto rows_prefetch = [&](int sub, int b) {
          l4n = *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)(lseoff + (32 * sub + 8 * b + BUF * BQ) * 4);
        };
        // the dP accumulator of a sub-block starts as D (V is held negated: it ends as D - dP)
        auto init_dp = [&](Sub& x, int sub) {
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const f32x4 t = *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)(dvoff + (32 * sub + 8 * b + BUF * BQ) * 4);
#pragma unroll
            for (int v = 0; v < 4; ++v) x.dp[4 * b + v] = t[v];
          }
        };
        auto stage2 = [&](Sub& x, int sub, int i, float e_val, auto masked) {
          const int b = i >> 2, v = i & 3;
          float pr = e_val;
          if (decltype(masked)::value) {
            const int q_in = qb + 32 * sub + 8 * b + 4 * hh + v;
            if (key_in > q_in || q_in >= s_len) pr = 0.f;
          }
          const float ds = pr * x.dp[i];
          if (i & 1) {
            x.pb[b >> 1].w[2 * (b & 1) + (v >> 1)] = pack_bf16(pr_even, pr);
            x.dsb[b >> 1].w[2 * (b & 1) + (v >> 1)] = pack_bf16(ds_even, ds);
          } else {
            pr_even = pr;
            ds_even = ds;
          }
        };
        // slices 0..16: slice i runs stage 1 of element i (i < 16) and stage 2 of element i-1 (i > 0)
        auto sm_slice = [&](Sub& x, int sub, int i, auto masked) {
          const float e_prev = e_cur;
          if (i < 16) {
            const int b = i >> 2, v = i & 3;
            if (v == 0) {
              l4 = l4n;
              if (b < 3) rows_prefetch(sub, b + 1);
            }
            e_cur = __builtin_amdgcn_exp2f(__builtin_fmaf(x.s[i], p.scale_log2, -l4[v]));
          }
          if (i > 0) stage2(x, sub, i - 1, e_prev, masked);
        };
        // Every update of the dK^T / dV^T accumulators of a step is issued from ONE place (the two gr
        // chains at the end), whatever path computed the probabilities: with updates in several
        // branches the compiler keeps a second set of the 128 accumulator registers and copies one
        // set to the other in every step (one vector instruction per register).
        //
        // The step opens with the first LDS reads of sub-block A, which depend on nothing but the buffer: a
        // single wave per SIMD has nothing else to run while they are under way, so everything that can wait
        // (the step's flags, the copies for the next step) comes after them, and the copies go out one by one
        // behind the first MFMA chain, which carries no vector arithmetic (measured per step of 3600 clocks:
        // 800 clocks from the last MFMA of a step to the first of the next with the bookkeeping, a burst of
        // copies and the reads one after the other; 350 this way, and the copies cost the chain 340).
        Sub xa, xb;
        LdsChain<NC + NCV, kPD> c1;
        c1.prefill(sd_load(0));
        init_dp(xa, 0);  // behind the operand reads: only the first dP MFMA needs it
        // not in reach: the block lies above this wave's keys, or this is the idle step that makes the count even
        const bool in_reach = wave_active && active && qb + BQ - 1 >= kw0_in;
        const bool need_a = in_reach && qb + 31 >= kw0_in;           // qb < s_len always holds
        const bool need_b = in_reach && qb + 63 >= kw0_in && qb + 32 < s_len;
        const bool any_mask = kw0_in + 31 > qb || qb + 63 >= s_len;  // diagonal or sample tail in reach
        const bool pair = need_a && need_b && !any_mask;
        if (pair) {
          // a next block with all its rows (every block but a sample's last) is copied slot by slot behind
          // the MFMAs; the clamped form needs vector arithmetic and registers, and goes out up front.  One
          // chain for both cases: with the chain on two paths the compiler joins the score registers by
          // copies placed right behind the asm MFMAs, before their results exist.
          const bool behind = has_next && next_is_full();
          if (has_next && !behind) issue_next(1 - BUF);
          c1.template run_with<N_COPY>(sd_load(0), sd_mma(xa), [&](int slot) {
            if (behind) issue_copy(slot, 1 - BUF, std::true_type{});
          });
          rows_prefetch(0, 0);
          init_dp(xb, 1);
          c1.prefill(sd_load(1));
          if (kVgprScores) mfma_results_ready(xa.s, xa.dp);
          c1.template run_with<16>(sd_load(1), sd_mma(xb), [&](int i) { sm_slice(xa, 0, i, std::false_type{}); });
          sm_slice(xa, 0, 16, std::false_type{});
        } else {
          // sub-block A: masked, finished here.  Sub-block B: its probabilities are formed by the same
          // unmasked slices as on the fast path (behind the first gr chain below), so the mask goes
          // into the scores instead: -inf gives exp2 = 0 (the scale is positive) and dS = 0 (dP - D).
          if (has_next) issue_next(1 - BUF);
          if (need_a) {
            c1.run(sd_load(0), sd_mma(xa));
            rows_prefetch(0, 0);
            if (kVgprScores) mfma_results_ready(xa.s, xa.dp);
#pragma unroll
            for (int i = 0; i < 17; ++i) sm_slice(xa, 0, i, std::true_type{});
          } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              xa.pb[j].u = u32x4{0, 0, 0, 0};
              xa.dsb[j].u = u32x4{0, 0, 0, 0};
            }
          }
          if (need_b) {
            init_dp(xb, 1);
            c1.prefill(sd_load(1));
            c1.run(sd_load(1), sd_mma(xb));
            if (kVgprScores) mfma_results_ready(xb.s, xb.dp);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int q_in = qb + 32 + 8 * (i >> 2) + 4 * hh + (i & 3);
              if (key_in > q_in || q_in >= s_len) xb.s[i] = -INFINITY;
            }
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              xb.s[i] = -INFINITY;
              xb.dp[i] = 0.f;
            }
          }
        }
        rows_prefetch(1, 0);
        __builtin_amdgcn_sched_barrier(0);
        LdsChain<2 * NEB + 2 * NDB, kPD> c2;
        c2.prefill(gr_load(0));
        if (kVgprScores) mfma_results_ready(xb.s, xb.dp);
        c2.template run_with<16>(gr_load(0), gr_mma(xa), [&](int i) { sm_slice(xb, 1, i, std::false_type{}); });
        sm_slice(xb, 1, 16, std::false_type{});
        c2.prefill(gr_load(1));
        c2.run(gr_load(1), gr_mma(xb));
      };

      // Two steps per iteration, one on each buffer, with no branch between them: the accumulators are
      // updated at two places that follow each other, never on alternative paths.  An odd number of
      // steps is rounded up by an idle step (zero operands).
      for (int step = 0; step < n_steps; step += 2) {
        wait_async_loads();
        __syncthreads();
        do_step(std::integral_constant<int, 0>{}, true, step + 1 < n_steps);
        race_fence();
        wait_async_loads();
        __syncthreads();
        do_step(std::integral_constant<int, 1>{}, step + 1 < n_steps, step + 2 < n_steps);
        race_fence();
      }

      if (p.n_split == 1) {
        if (wave_active) {  // both through the wave's rows of K
          RowStage<DQK>::put(k_at, lane, dkt, -p.scale);
          RowStage<DQK>::copy_out(p.dk + (int64_t)first_key * p.k_st + (int64_t)kh * p.k_sh, (uint32_t)p.k_st * 2, tl.row_end - first_key, k_at, lane);
          RowStage<DV>::put(k_at, lane, dvt, 1.0f);
          RowStage<DV>::copy_out(p.dv + (int64_t)first_key * p.v_st + (int64_t)kh * p.v_sh, (uint32_t)p.v_st * 2, tl.row_end - first_key, k_at, lane);
        }
      } else if (key_valid) {
        // this part's sums, fp32, [part][key][kv head][dim]; the reduce kernel adds the parts up
        const int64_t row = ((int64_t)part * p.T + my_key) * p.Hkv + kh;
        float* dkp = p.dk_part + row * DQK + 4 * hh;
        float* dvp = p.dv_part + row * DV + 4 * hh;
        const float ksc = -p.scale;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            *(f32x4*)(dkp + 32 * db + 8 * b) = f32x4{dkt[db][4 * b] * ksc, dkt[db][4 * b + 1] * ksc,
                                                       dkt[db][4 * b + 2] * ksc, dkt[db][4 * b + 3] * ksc};
#pragma unroll
        for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            *(f32x4*)(dvp + 32 * eb + 8 * b) = f32x4{dvt[eb][4 * b], dvt[eb][4 * b + 1], dvt[eb][4 * b + 2], dvt[eb][4 * b + 3]};
      }
    }
    prof_end(pa, profiled, tid);
    if constexpr (DIRECT) break;
  }
  prof_write(pa, profiled, bwd_args<false>()->prof, tid);
}
template <int DQK, int DV>
__global__ __launch_bounds__(kThreads, 1) void bwd_dkdv_kernel(const BwdParams) {
  dkdv_items<DQK, DV>(0, (int)gridDim.x);
}
// dK/dV and dQ in one launch at head size 192: workgroups of four wavefronts, an item of either each, dK/dV first (as
// many dQ items as dK/dV: in turn they would keep to half of a die's shader engines each).
template <int DQK, int DV>
__global__ __launch_bounds__(kThreads, 1) void bwd_both4_kernel(const BwdParams, int n_dkdv, int n_resident) {
  if ((int)blockIdx.x < n_dkdv) dkdv_items<DQK, DV, true>((int)blockIdx.x, n_resident);
  else dq_items<DQK, DV, 1, false, true>((int)blockIdx.x - n_dkdv);
}

// ------------------------------------------------------------------- dK, dV, eight wavefronts
// The same items with two wavefronts per SIMD, head sizes 64 and 128: two groups of four wavefronts.  Wave kg of either
// group holds the dK^T / dV^T accumulators of keys 32 kg .. 32 kg + 31; group 0 takes the first 32 rows of every block
// of 64 query rows, group 1 the last.  At the end of an item each of the two waves of a key group hands one of its two
// accumulators to the other through LDS and finishes the other one.
//
// A lone wave per SIMD (the kernel above) issues one instruction every 5 to 6 clocks, and a step has about 6 an MFMA:
// it is bound by its own instruction stream, the matrix pipe 57 % busy.  Two waves of half the rows fill each other's
// gaps: 67 % busy, 16 % fewer clocks a launch (32768 tokens with a sample of 16384; 70 % at 131072 tokens).  That makes the
// launch only 3 to 5 % shorter, since the card, at its power limit, then clocks 1.74 GHz instead of 1.93; the fewer clocks
// of a step matter most where it is not.  What makes room
// for the second wave in 256 registers a lane: the scores of 32 rows alone in flight, their own four stages following
// each other (S | dP and the probabilities | dV and dS | dK), and at head size 128 the K fragments read from LDS in
// every step.  dK/dV kernel, four waves -> eight, us: 8192 tokens, 32/8 heads of 128: 184 -> 159; 32768 tokens with a
// sample of 16384: 4062 -> 3869, 8/1 heads 1067 -> 1039; 131072 tokens, 64/8 heads, ms: 291 -> 277; 5497 tokens, 8 heads
// of 64: 49.3 -> 42.5; 1024 tokens, 4 heads of 64: 14.8 -> 13.5.
// The exchange at the end costs an item 1.9 us: see eight_waves() for where the line lies.
//
// At head size 128 it spills 5 vector and 35 scalar registers: 32 bytes of scratch a lane, none of it touched between the
// first and the last MFMA, and two reads of a spilled scalar in three steps.
//
// K and V come in whole rows through LDS and dK and dV go out that way (RowStage).  A row a lane, the 12 loads of eight
// wavefronts hold the address path 64 clocks each, 6144 of an item, and their 8 stores 4096; in whole rows a quarter of it.
//
// Tried here and slower or the same: V in LDS too (the LDS pipe, busy in half the clocks, costs power: +2 %); the two
// groups half a step apart (+2 %); s_setprio around the MFMA chains; copies with a wait of their own in mid-step.
//
// DIRECT: the launch's item `block` and no other (see bwd_both_kernel).  n_resident: workgroups under way at a time.
template <int DQK, int DV, bool DIRECT = false>
__device__ __forceinline__ void dkdv8_items(int block, int n_resident) {
  static_assert(DQK == DV, "one set of lane offsets for Q and dO");
  constexpr int BN = 128, BQ = 64, SUB = 32, NBUF = 3;
  constexpr int QRB = DQK * 2;
  constexpr int TILE = SUB * QRB, PAIR = 2 * TILE;  // Q and dO of a step, one group
  constexpr int NC = DQK / 16, NDB = DQK / 32;
  constexpr bool kKLds = DQK > 64;  // K fragments read from LDS in every step
  // K fragments, and in front of an item's first step the tile's rows of K; those of V where the third buffers are
  constexpr int K_AT = 2 * NBUF * PAIR, ROWS_AT = K_AT + 4 * RowStage<DQK>::BYTES;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // [group][buffer][Q | dO], [K fragments], [group][buffer][64 LSE2 | 64 D | 128 of no use]
  // (32 used of each 64: a copy by 64 lanes writes zeros behind its rows)
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qs = wave >> 2, share = DQK > 64 ? mirrored(wave) : wave, kg = share & 3;
  const int lane = tid & 63, l32 = lane & 31, hh = lane >> 5;

  const uint32_t lds0 = lds_address(smem);
  uint32_t qoff[NC], qtoff[2][NDB];
#pragma unroll
  for (int c = 0; c < NC; ++c) qoff[c] = lds0 + qs * (NBUF * PAIR) + l32 * QRB + swz<DQK>(2 * c + hh, l32) * 16;
  {
    const int G = lane >> 4, s = lane & 15;
    const int k8 = 4 * hh + (s >> 2);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const int c = 4 * db + 2 * (G & 1) + ((s & 3) >> 1);
        qtoff[r][db] = lds0 + qs * (NBUF * PAIR) + (8 * r + k8) * QRB + swz<DQK>(c, 8 * r + k8) * 16 + (s & 1) * 8;
      }
  }
  const uint32_t kfoff = lds0 + K_AT + kg * (NC * 1024) + lane * 16;
  uint32_t lseoff = lds0 + ROWS_AT + qs * (NBUF * 1024) + 16 * hh;
  // opaque: the compiler would otherwise rebuild some of these from each other in front of their reads
  asm volatile("" : "+v"(lseoff));
#pragma unroll
  for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(qoff[c]));
#pragma unroll
  for (int db = 0; db < NDB; ++db) asm volatile("" : "+v"(qtoff[0][db]), "+v"(qtoff[1][db]));
  const uint32_t tiles = lds0 + qs * (NBUF * PAIR) + kg * 1024, rows_lds = lds0 + ROWS_AT + qs * (NBUF * 1024) + kg * 256;

  const uint32_t q_stride_b = (uint32_t)bwd_args<false>()->q_st * 2, o_stride_b = (uint32_t)bwd_args<false>()->o_st * 2;
  FullTileLoader<DQK, SUB> q_loader, o_loader;
  q_loader.init(kg, lane, q_stride_b);
  o_loader.init(kg, lane, o_stride_b);

  const bool profiled = !DIRECT && bwd_args<false>()->prof;
  ProfAcc pa;
  int q_cur = xcc_id_reg() & (kNumXcd - 1), q_tried = 0;
  for (;;) {
    const BwdArgs& p = *bwd_args<!DIRECT>();
    const WorkQueues wq{p.counter, p.n_tiles, p.Hkv * p.n_split, 1};
    const int g_item = quotient(p.g, p.n_split);
    int tile_idx, vh;
    if constexpr (DIRECT) {
      const Taken tk = direct_item_inline(wq.n_tiles, wq.Hkv, 1, 0, 0, block);
      tile_idx = __builtin_amdgcn_readfirstlane(tk.tile_idx);
      vh = __builtin_amdgcn_readfirstlane(tk.head);
    } else {
      if (!next_item(wq, (int*)smem, tid, q_cur, q_tried, tile_idx, vh)) break;
    }
    const int kh = quotient(vh, p.n_split), part = vh - kh * p.n_split;
    const int head0 = vh * g_item;
    prof_begin(pa, profiled, wave);

    hbp_tile tl;
    int s0, s1;
    bool ok = load_tile(p.tiles, tile_idx, p.cu, p.n_samples, lane, tl, s0, s1);
    if (ok) {
      ok = s0 >= 0 && s1 <= p.T && s0 <= tl.row_begin && tl.row_begin < tl.row_end &&
           tl.row_end <= s1 && tl.row_end - tl.row_begin <= BN;
    }
    if (ok) {
      const int s_len = s1 - s0;
      const int k0_in = tl.row_begin - s0;
      const int kw0_in = k0_in + 32 * kg;
      const int my_key = tl.row_begin + 32 * kg + l32;
      const bool key_valid = my_key < tl.row_end;
      const bool wave_active = tl.row_begin + 32 * kg < tl.row_end;

      const int qb_start = (k0_in / BQ) * BQ;
      const int nqb = (s_len - qb_start + BQ - 1) / BQ;
      const int n_steps = nqb * g_item;
      const int w_share = quotient(n_resident, min(p.Hkv * p.n_split, kNumXcd * kHeadGroup));
      const int set = quotient(tl.tile, max(w_share, 1));
      int skip = w_share >= 8 && (set & 1) ? (tl.tile - set * w_share) * (BN / BQ) : 0;
      skip = max(0, min(skip, nqb - 1));
      // Step order as in the four-wave kernel.  The copies of a step's operands run two steps ahead, one by one behind the
      // updates: their address path takes 16 clocks of the compute unit a copy, and a burst of them holds the waves.  State of the copying side: the block and head of the next
      // step to copy, its first row of this group's 32 (in-sample), the steps left, and the descriptors of the three
      // sources (Q, dO, and LSE2 or D: waves 0 and 1 of a group copy those).
      int blk_next = nqb - 1 - skip, head_next = 0, copies_left = n_steps;
      int q0_next = qb_start + blk_next * BQ + SUB * qs;
      u32x4 q_desc, o_desc, r_desc;
      auto set_spans = [&]() {
        const int rows = copies_left > 0 ? s_len - q0_next : 0;
        q_desc[2] = rows_span(rows, SUB, q_stride_b, QRB);
        o_desc[2] = rows_span(rows, SUB, o_stride_b, QRB);
        r_desc[2] = kg < 2 ? rows_span(rows, SUB, 4, 4) : 0;
      };
      {
        const int64_t row = (int64_t)s0 + q0_next;
        q_desc = buffer_desc(p.q + row * p.q_st + (int64_t)head0 * p.q_sh, 0);
        o_desc = buffer_desc(p.d_o + row * p.o_st + (int64_t)head0 * p.o_sh, 0);
        r_desc = buffer_desc((kg == 0 ? p.lse2 : p.D) + (int64_t)head0 * p.T + row, 0);
        set_spans();
      }
      constexpr int NQC = decltype(q_loader)::PER_WAVE, N_COPY = 2 * NQC + 1;
      int q0_in[NBUF] = {0, 0, 0};
      auto issue_copy = [&](auto slot_tag, auto buf_tag) {
        constexpr int SLOT = decltype(slot_tag)::value, BUF = decltype(buf_tag)::value;
        if constexpr (SLOT < NQC) buffer_copy16<BUF * PAIR + SLOT * 4096>(q_desc, q_loader.off[SLOT], tiles);
        else if constexpr (SLOT < 2 * NQC) buffer_copy16<BUF * PAIR + TILE + (SLOT - NQC) * 4096>(o_desc, o_loader.off[SLOT - NQC], tiles);
        else buffer_copy4<BUF * 1024>(r_desc, lane * 4, rows_lds);
      };
      // to the first head of the block before, from the last head of a block
      const int64_t q_blk = -2 * ((int64_t)BQ * p.q_st + (int64_t)(g_item - 1) * p.q_sh);
      const int64_t o_blk = -2 * ((int64_t)BQ * p.o_st + (int64_t)(g_item - 1) * p.o_sh);
      const int64_t r_blk = -4 * ((int64_t)BQ + (int64_t)(g_item - 1) * p.T);
      auto advance = [&](int buf) {
        q0_in[buf] = q0_next;
        --copies_left;
        if (++head_next < g_item) {
          buffer_advance(q_desc, 2 * p.q_sh);
          buffer_advance(o_desc, 2 * p.o_sh);
          buffer_advance(r_desc, 4 * (int64_t)p.T);
        } else {
          head_next = 0;
          buffer_advance(q_desc, q_blk);
          buffer_advance(o_desc, o_blk);
          buffer_advance(r_desc, r_blk);
          q0_next -= BQ;
          if (--blk_next < 0) {  // on from the tile's own block to the sample's last
            blk_next += nqb;
            q0_next += nqb * BQ;
            buffer_advance(q_desc, 2 * (int64_t)nqb * BQ * p.q_st);
            buffer_advance(o_desc, 2 * (int64_t)nqb * BQ * p.o_st);
            buffer_advance(r_desc, 4 * (int64_t)nqb * BQ);
          }
          // only the sample's last block may have fewer rows; and none are copied behind the item's last step
          if (blk_next >= nqb - 2 || copies_left <= 0) set_spans();
        }
      };
      auto issue_all = [&](auto buf_tag) {
        issue_copy(std::integral_constant<int, 0>{}, buf_tag);
        issue_copy(std::integral_constant<int, 1>{}, buf_tag);
        issue_copy(std::integral_constant<int, 2>{}, buf_tag);
        if constexpr (N_COPY > 3) issue_copy(std::integral_constant<int, 3>{}, buf_tag);
        if constexpr (N_COPY > 4) issue_copy(std::integral_constant<int, 4>{}, buf_tag);
      };
      static_assert(N_COPY == 3 || N_COPY == 5, "32 rows of 128 or 256 bytes on four waves");
      // K and V in whole rows (RowStage), half of a key group's by either of its waves
      const uint32_t k_at = lds0 + K_AT + kg * RowStage<DQK>::BYTES;
      const uint32_t v_at = lds0 + (kg >> 1) * (NBUF * PAIR) + 2 * PAIR + (kg & 1) * RowStage<DQK>::BYTES;
      const int first_key = tl.row_begin + 32 * kg, keys_left = tl.row_end - first_key;
      RowStage<DQK>::template copy_in<2>(p.k + (int64_t)first_key * p.k_st + (int64_t)kh * p.k_sh, (uint32_t)p.k_st * 2, keys_left, k_at, lane, qs);
      RowStage<DQK>::template copy_in<2>(p.v + (int64_t)first_key * p.v_st + (int64_t)kh * p.v_sh, (uint32_t)p.v_st * 2, keys_left, v_at, lane, qs);
      issue_all(std::integral_constant<int, 0>{});
      advance(0);
      issue_all(std::integral_constant<int, 1>{});
      advance(1);
      wait_async_but<2 * N_COPY>();
      race_fence();
      __syncthreads();

      Frag knat[NC], vnat[NC];
      {
        RowStage<DQK>::fragments(k_at, lane, knat);
        RowStage<DQK>::fragments(v_at, lane, vnat);
        race_fence();
        if constexpr (kKLds) {  // the two waves of a key group write half of the fragments each, where the rows were
          lds_barrier();
#pragma unroll
          for (int c = 0; c < NC / 2; ++c)
            *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(kfoff + (2 * c + qs) * 1024) = qs ? knat[2 * c + 1].u : knat[2 * c].u;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) vnat[c].u ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
      }
      f32x16 dkt[NDB], dvt[NDB];
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dkt[db][i] = dvt[db][i] = 0.f;

      constexpr int kPD = 3;
      auto pin = [](auto& x) {  // keeps a slice's result where it is computed: it is used behind the next chain
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+v"(x));
#endif
      };
      const int kw0 = wave_active ? kw0_in : 0x7fffffe0;  // no block is in reach of an idle wave
      // The copies of the step after next go to the buffer that the step before this one has left.
      auto do_step = [&](auto buf_tag) {
        constexpr int BUF = decltype(buf_tag)::value, CBUF = (BUF + 2) % NBUF;
        const std::integral_constant<int, CBUF> cbuf{};
        __builtin_amdgcn_s_waitcnt(0x0F70 + N_COPY);  // all copies but the last step's, which are the next step's operands
        __syncthreads();
        const int q0 = q0_in[BUF];
        const bool need = ((q0 + 31 - kw0) | (s_len - 1 - q0)) >= 0;  // not above this wave's keys, nor behind the sample
        typedef const __attribute__((address_space(3))) u32x4* lds_u4;
        typedef const __attribute__((address_space(3))) f32x4* lds_f4;
        auto q_load = [&](int i) { Frag a; a.u = *(lds_u4)(uintptr_t)(qoff[i] + BUF * PAIR); return a; };
        auto o_load = [&](int i) { Frag a; a.u = *(lds_u4)(uintptr_t)(qoff[i] + (BUF * PAIR + TILE)); return a; };
        auto k_load = [&](int i) { Frag a; a.u = *(lds_u4)(uintptr_t)(kfoff + i * 1024); return a; };
        auto t_load = [&](int i, int base) {
          const int db = i % NDB, j = i / NDB;
          Frag a;
          a.h[0] = lds_read_tr16_at(qtoff[0][db] + (16 * j * QRB + base));
          a.h[1] = lds_read_tr16_at(qtoff[1][db] + (16 * j * QRB + base));
          return a;
        };
        if (need) {
          f32x16 s, dp;
          Frag pb[2], dsb[2];
          // ---- S = Q K^T
          Frag rq[kPD], rk[kPD];
#pragma unroll
          for (int i = 0; i < kPD; ++i) {
            rq[i] = q_load(i);
            if constexpr (kKLds) rk[i] = k_load(i);
          }
#pragma unroll
          for (int b = 0; b < 4; ++b) {  // D of the rows: dP starts there (V is held negated: it ends as D - dP)
            const f32x4 t = *(lds_f4)(uintptr_t)(lseoff + BUF * 1024 + 256 + 32 * b);
#pragma unroll
            for (int v = 0; v < 4; ++v) dp[4 * b + v] = t[v];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < NC; ++i) {
            const bf16x8 kb = kKLds ? rk[i % kPD].v : knat[i].v;
            if (i == 0) s = mfma32_vgpr_first(rq[0].v, kb);
            else mfma32_vgpr(s, rq[i % kPD].v, kb);
            if (i + kPD < NC) {
              rq[i % kPD] = q_load(i + kPD);
              if constexpr (kKLds) rk[i % kPD] = k_load(i + kPD);
            } else {
              rq[i % kPD] = o_load(i + kPD - NC);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          // ---- dP = dO V^T, the probabilities behind it
          f32x4 l4 = *(lds_f4)(uintptr_t)(lseoff + BUF * 1024), l4n;
          mfma32_vgpr(dp, rq[NC % kPD].v, vnat[0].v);
          rq[NC % kPD] = o_load(kPD);
          mfma_result_ready(s);
          if (((q0 - kw0_in - 31) | (s_len - 32 - q0)) < 0) {  // the diagonal or the sample's end in reach
            int x = lane;  // opaque: rebuilt here, not held across the loop
            asm volatile("" : "+v"(x));
            const int e0 = q0 + 4 * (x >> 5);
            int d = kw0_in + (x & 31) - e0, e = s_len - e0;  // row 8b + 4hh + v: masked below d and from e on
            asm volatile("" : "+v"(d), "+v"(e));
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (8 * (i >> 2) + (i & 3) < d || 8 * (i >> 2) + (i & 3) >= e) s[i] = -INFINITY;
          }
          __builtin_amdgcn_sched_barrier(0);
          auto p_slice = [&](int i) {  // 0..16: exp of element i, pack of the pair that ends at element i - 1
            if (i < 16) {
              const int b = i >> 2, v = i & 3;
              if (v == 0) {
                if (i) l4 = l4n;
                if (b < 3) l4n = *(lds_f4)(uintptr_t)(lseoff + BUF * 1024 + 32 * (b + 1));
              }
              float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], p.scale_log2, -l4[v]));
              pin(e);
              s[i] = e;
            }
            if (i > 0 && (i & 1) == 0) {
              const int e = i - 2;
              pb[e >> 3].w[(e & 7) >> 1] = pack_bf16(s[e], s[e + 1]);
              pin(pb[e >> 3].w[(e & 7) >> 1]);
            }
          };
          constexpr int LP = NC - 1;
#pragma unroll
          for (int i = 1; i < NC; ++i) {
            mfma32_vgpr(dp, rq[(NC + i) % kPD].v, vnat[i].v);
            if (i + kPD < NC) rq[(NC + i) % kPD] = o_load(i + kPD);
#pragma unroll
            for (int sl = (i - 1) * 17 / LP; sl < i * 17 / LP; ++sl) p_slice(sl);
            __builtin_amdgcn_sched_barrier(0);
          }
          // ---- dV^T += dO^T P, dS behind it; dK^T += Q^T dS
          Frag rt[kPD];
          auto g_load = [&](int i) { return i < 2 * NDB ? t_load(i, BUF * PAIR + TILE) : t_load(i - 2 * NDB, BUF * PAIR); };
#pragma unroll
          for (int i = 0; i < kPD; ++i) rt[i] = g_load(i);
          __builtin_amdgcn_sched_barrier(0);
          mfma_result_ready(dp);
          constexpr int LG = 4 * NDB, LV = 2 * NDB, GAP = LG / N_COPY;
          auto copy_behind = [&](auto slot_tag, int i) {
            constexpr int SLOT = decltype(slot_tag)::value;
            if constexpr (SLOT < N_COPY)
              if (i == 1 + SLOT * GAP) issue_copy(slot_tag, cbuf);
          };
#pragma unroll
          for (int i = 0; i < LG; ++i) {
            const int db = i % NDB, j = (i / NDB) & 1;
            if (i < LV) dvt[db] = mfma32(rt[i % kPD].v, pb[j].v, dvt[db]);
            else dkt[db] = mfma32(rt[i % kPD].v, dsb[j].v, dkt[db]);
            if (i + kPD < LG) rt[i % kPD] = g_load(i + kPD);
            if (i < LV) {
#pragma unroll
              for (int e = i * 8 / LV * 2; e < (i + 1) * 8 / LV * 2; e += 2) {
                dsb[e >> 3].w[(e & 7) >> 1] = pack_bf16(s[e] * dp[e], s[e + 1] * dp[e + 1]);
                pin(dsb[e >> 3].w[(e & 7) >> 1]);
              }
            }
            copy_behind(std::integral_constant<int, 0>{}, i);
            copy_behind(std::integral_constant<int, 1>{}, i);
            copy_behind(std::integral_constant<int, 2>{}, i);
            copy_behind(std::integral_constant<int, 3>{}, i);
            copy_behind(std::integral_constant<int, 4>{}, i);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          issue_all(cbuf);
        }
        advance(CBUF);
        race_fence();
      };

      for (int step = 0; step < n_steps; step += 3) {
        do_step(std::integral_constant<int, 0>{});
        if (step + 1 < n_steps) do_step(std::integral_constant<int, 1>{});
        if (step + 2 < n_steps) do_step(std::integral_constant<int, 2>{});
      }
      wait_async_loads();

      // The two waves of a pair: the upper rows' wave hands over its dK^T and finishes dV, the other the reverse.
      __syncthreads();  // the tile buffers are no longer read
      const uint32_t mine = lds0 + share * (NDB * 4096) + lane * 16, theirs = lds0 + (share ^ 4) * (NDB * 4096) + lane * 16;
      typedef __attribute__((address_space(3))) f32x4* lds_w4;
      auto send = [&](const f32x16 (&acc)[NDB]) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            *(lds_w4)(uintptr_t)(mine + (4 * db + b) * 1024) = f32x4{acc[db][4 * b], acc[db][4 * b + 1], acc[db][4 * b + 2], acc[db][4 * b + 3]};
      };
      auto receive = [&](f32x16 (&acc)[NDB]) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const f32x4 t = *(const __attribute__((address_space(3))) f32x4*)(uintptr_t)(theirs + (4 * db + b) * 1024);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[db][4 * b + v] += t[v];
          }
      };
      auto store = [&](const f32x16 (&acc)[NDB], uint16_t* out, int64_t st, int64_t sh, float* parts, float scale) {
        if (p.n_split == 1) {
          if (wave_active) {  // through what this wave alone has read
            const uint32_t at = theirs - lane * 16;
            RowStage<DQK>::put(at, lane, acc, scale);
            RowStage<DQK>::copy_out(out + (int64_t)first_key * st + (int64_t)kh * sh, (uint32_t)st * 2, keys_left, at, lane);
          }
        } else if (key_valid) {
          float* row = parts + (((int64_t)part * p.T + my_key) * p.Hkv + kh) * DQK + 4 * hh;
#pragma unroll
          for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int b = 0; b < 4; ++b)
              *(f32x4*)(row + 32 * db + 8 * b) = f32x4{acc[db][4 * b] * scale, acc[db][4 * b + 1] * scale,
                                                         acc[db][4 * b + 2] * scale, acc[db][4 * b + 3] * scale};
        }
      };
      if (qs == 0) send(dkt);
      else send(dvt);
      __syncthreads();
      if (qs == 0) {
        receive(dvt);
        store(dvt, p.dv, p.v_st, p.v_sh, p.dv_part, 1.0f);
      } else {
        receive(dkt);
        store(dkt, p.dk, p.k_st, p.k_sh, p.dk_part, -p.scale);
      }
    }
    prof_end(pa, profiled, wave);
    if constexpr (DIRECT) break;
  }
  prof_write(pa, profiled, bwd_args<false>()->prof, tid);
}
template <int DQK, int DV>
__global__ __launch_bounds__(2 * kThreads, 2) void bwd_dkdv8_kernel(const BwdParams) {
  dkdv8_items<DQK, DV>(0, (int)gridDim.x);
}

// dK/dV and dQ in one launch, for packs of few rounds: neither needs the other, and with two launches the chip is partly
// idle at the end of each (a dK/dV item is as long as its sample, and the second launch waits for the last one).  Every
// workgroup takes one item, dispatched in order, without queues: a dK/dV item, or dQ of one tile for two query heads.
// interleave = 0: dK/dV first (its items are the longer ones), then dQ.  interleave = 1: both worklists (longest first)
// in proportion, eight workgroups, one a die, at a time; so the launch ends with the shortest items of both and not with
// all of dQ.  Measured lines and gains: see one_launch().
// Tried and dropped: dQ in pairs of heads in a launch of its own with queues (.86 to 1.02 of the present one's speed).
template <int DQK, int DV, bool SHARED>
__global__ __launch_bounds__(2 * kThreads, 2) void bwd_both_kernel(const BwdParams, int n_dkdv, int n_dq, int n_resident,
                                                                   int interleave) {
  bool is_dkdv = (int)blockIdx.x < n_dkdv;
  int block = is_dkdv ? (int)blockIdx.x : (int)blockIdx.x - n_dkdv;
  if (interleave) {  // of the first k groups of eight, ceil(k groups_dkdv / groups) are dK/dV
    const uint32_t groups_dkdv = (uint32_t)(n_dkdv + kNumXcd - 1) / kNumXcd;
    const uint32_t groups = groups_dkdv + (uint32_t)(n_dq + kNumXcd - 1) / kNumXcd, k = blockIdx.x / kNumXcd;
    const uint32_t in_front = quotient(k * groups_dkdv + groups - 1, groups);
    is_dkdv = quotient((k + 1) * groups_dkdv + groups - 1, groups) > (int)in_front;
    block = (int)(kNumXcd * (is_dkdv ? in_front : k - in_front) + blockIdx.x % kNumXcd);
    if (block >= (is_dkdv ? n_dkdv : n_dq)) return;
  }
  if (is_dkdv) dkdv8_items<DQK, DV, true>(block, n_resident);
  else dq_items<DQK, DV, 2, SHARED>(block);
}

// dK, dV = sum over the parts of the partial sums of the key-tile kernel, in part order.  Workgroups (x, y):
// share y of key tile x of the worklist (only rows covered by a tile are written, as without parts); a thread
// handles four consecutive dims of one (key, kv head) at a time.  HBM-bound: every partial sum is read once.
// With one workgroup a tile there were too few loads under way; with kReduceUnits units a thread, T = 32768:
// 8 parts (8/1 heads) 135 -> 57 us, 5.0 TB/s; 4 parts (12/3) 184 -> 93, 4.9; 3 (6/2, d = 64) 30 -> 19, 6.1;
// 2 (32/4) 112 -> 60, 5.6; T = 4096, 4 parts: 97 -> 10.  Four loads of a thread are under way from five parts
// on; with fewer a thread waits for each of its one to three, and the many workgroups make up for it.
constexpr int kReduceUnits = 2;
template <int DQK, int DV>
__global__ __launch_bounds__(kThreads) void bwd_reduce_parts_kernel(const BwdParams p) {
  const hbp_tile tl = p.tiles[blockIdx.x];
  if (tl.sample < 0 || tl.sample >= p.n_samples) return;
  const int s0 = p.cu[tl.sample], s1 = p.cu[tl.sample + 1];
  if (!(s0 >= 0 && s1 <= p.T && s0 <= tl.row_begin && tl.row_begin < tl.row_end && tl.row_end <= s1 &&
        tl.row_end - tl.row_begin <= 128))
    return;
  constexpr uint32_t QK4 = DQK / 4, V4 = DV / 4;
  const uint32_t n_heads = p.Hkv, n_units = (uint32_t)(tl.row_end - tl.row_begin) * n_heads * (QK4 + V4);
  for (uint32_t u = blockIdx.y * kThreads + threadIdx.x; u < n_units; u += gridDim.y * kThreads) {
    const uint32_t c = u % (QK4 + V4), rk = u / (QK4 + V4);
    const uint32_t row = rk / n_heads, kh = rk - row * n_heads;
    const int64_t key = tl.row_begin + row;
    const bool is_k = c < QK4;
    const int dim = is_k ? DQK : DV, x = 4 * (is_k ? c : c - QK4);
    const float* src = (is_k ? p.dk_part : p.dv_part) + (key * p.Hkv + kh) * dim + x;
    const int64_t part_stride = (int64_t)p.T * p.Hkv * dim;
    f32x4 acc = *(const f32x4*)src;
    int part = 1;
    for (; part + 4 <= p.n_split; part += 4) {  // four loads under way
      f32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *(const f32x4*)(src + (part + i) * part_stride);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc += v[i];
    }
    for (; part < p.n_split; ++part) acc += *(const f32x4*)(src + part * part_stride);
    uint16_t* dst = is_k ? p.dk + key * p.k_st + (int64_t)kh * p.k_sh + x : p.dv + key * p.v_st + (int64_t)kh * p.v_sh + x;
    *(u32x2*)dst = u32x2{pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3])};
  }
}

size_t bwd_partial_floats(int T, int Hkv, int g, int dim) {
  const int n_split = heads_split(Hkv, g);
  return n_split > 1 ? (size_t)n_split * (size_t)T * (size_t)Hkv * (size_t)dim : 0;
}

// D[h,r] = sum_x dO[r,h,x] O[r,h,x], LSE2 = LSE*log2(e); resets both scheduler counters.  HBM-bound: O and dO are read
// once.  A workgroup takes PAIRS (row, head) pairs: 1 to 8 heads (the largest power of two up to Hq) of as many rows as
// make up the rest, DV / 8 lanes of 16 bytes a pair.  Eight passes' loads are under way at a time, and the lanes' sums are
// added up through LDS by a thread a pair, which then has consecutive rows beside it: D, LSE and LSE2 in whole lines.
// With 256 pairs a workgroup against one part of a pair a thread (and 4-byte accesses), us: 8192 tokens, 32 heads of 128:
// 27.4 -> 24.2; 24 heads: 24.7 -> 16.8; 32768 tokens, 32 heads: 108 -> 99 (5.4 TB/s); 65536, 64 heads: 421 -> 395.  Up to
// kPreSmall pairs 64 a workgroup, or too few loads are under way: 2048 tokens, 32 heads: 7.96 -> 6.88 (256 pairs: 8.12).
constexpr int64_t kPreSmall = 131072;
inline int prepass_heads_log2(int Hq) { return Hq >= 8 ? 3 : Hq >= 4 ? 2 : Hq >= 2 ? 1 : 0; }
template <int DV, int PAIRS>
__global__ __launch_bounds__(kThreads) void bwd_prepass_kernel(const BwdParams p, int heads_log2) {
  constexpr int LPR = DV / 8, PER_PASS = kThreads / LPR, PASSES = PAIRS / PER_PASS, BATCH = PASSES < 8 ? PASSES : 8;
  constexpr int PAIRS_LOG2 = __builtin_ctz(PAIRS);
  static_assert(PAIRS <= kThreads && PAIRS % PER_PASS == 0 && PASSES % BATCH == 0, "a thread a pair at the end");
  __shared__ float sums[PAIRS * (LPR + 1)];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid < kNumXcd) {
    if (p.counter) p.counter[tid * kCounterStride] = 0;
    if (p.counter_dq) p.counter_dq[tid * kCounterStride] = 0;
  }
  const int heads = 1 << heads_log2, rows_log2 = PAIRS_LOG2 - heads_log2, rows = 1 << rows_log2;
  const int head_blocks = (p.Hq + heads - 1) >> heads_log2;
  const int h0 = (int)(blockIdx.x % (unsigned)head_blocks) << heads_log2;
  const int64_t r0 = (int64_t)(blockIdx.x / (unsigned)head_blocks) << rows_log2;
  const int part = tid % LPR;
#pragma unroll
  for (int first = 0; first < PASSES; first += BATCH) {
    u32x4 a[BATCH], b[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int pair = (first + i) * PER_PASS + tid / LPR;  // heads innermost
      const int64_t r = min(r0 + (pair >> heads_log2), (int64_t)p.T - 1);  // beyond the end: the last one, not stored
      const int h = min(h0 + (pair & (heads - 1)), p.Hq - 1);
      const int64_t off = r * p.o_st + (int64_t)h * p.o_sh + 8 * part;
      a[i] = __builtin_nontemporal_load((const u32x4*)(p.o + off));
      b[i] = *(const u32x4*)(p.d_o + off);
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int pair = (first + i) * PER_PASS + tid / LPR;
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += bf16_lo(a[i][k]) * bf16_lo(b[i][k]) + bf16_hi(a[i][k]) * bf16_hi(b[i][k]);
      sums[((((pair & (heads - 1)) << rows_log2) + (pair >> heads_log2)) * (LPR + 1)) + part] = acc;
    }
  }
  __syncthreads();
  if (PAIRS < kThreads && tid >= PAIRS) return;
  float s[LPR];
#pragma unroll
  for (int i = 0; i < LPR; ++i) s[i] = sums[tid * (LPR + 1) + i];
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1)
#pragma unroll
    for (int i = 0; i < m; ++i) s[i] += s[i + m];
  const int h = h0 + (tid >> rows_log2);
  const int64_t r = r0 + (tid & (rows - 1));
  if (h < p.Hq && r < p.T) {
    p.D[(int64_t)h * p.T + r] = s[0];
    p.lse2[(int64_t)h * p.T + r] = p.lse[(int64_t)h * p.T + r] * kLog2e;
  }
}

template <int DQK, int DV>
constexpr int dkdv8_lds() {
  constexpr int tiles = 2 * 3 * 32 * (DQK * 2 + DV * 2) + 128 * DQK * 2 + 2 * 3 * 1024;
  constexpr int sums = 8 * DQK / 32 * 4096;
  return tiles > sums ? tiles : sums;
}
template <int DQK, int DV>
static int launch_dkdv8(const BwdParams& p, int grid, hipStream_t s) {
  constexpr int lds = dkdv8_lds<DQK, DV>();
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)bwd_dkdv8_kernel<DQK, DV>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  hipLaunchKernelGGL((bwd_dkdv8_kernel<DQK, DV>), dim3(grid), dim3(2 * kThreads), lds, s, p);
  return 0;
}

template <int DQK, int DV, bool SHARED>
static int launch_both(BwdParams p, int n_resident, bool interleave, hipStream_t s) {
  constexpr int lds_dq = DqLds<DQK, DV, 2, SHARED>::BYTES, lds_dkdv = dkdv8_lds<DQK, DV>();
  constexpr int lds = lds_dq > lds_dkdv ? lds_dq : lds_dkdv;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)bwd_both_kernel<DQK, DV, SHARED>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  if (SHARED) p.n_split_dq = heads_split(p.Hkv, p.g / 2);  // its items are pairs of heads
  const int n_dkdv = p.n_tiles * p.Hkv * p.n_split, n_dq = p.n_q_tiles * ((p.Hq + 1) / 2);
  auto whole = [](int n) { return (n + kNumXcd - 1) / kNumXcd * kNumXcd; };
  const int grid = interleave ? whole(n_dkdv) + whole(n_dq) : n_dkdv + n_dq;
  hipLaunchKernelGGL((bwd_both_kernel<DQK, DV, SHARED>), dim3(grid), dim3(2 * kThreads), lds, s, p, n_dkdv, n_dq,
                     n_resident, (int)interleave);
  return (int)hipGetLastError();
}

template <int DQK, int DV>
static int launch_both4(const BwdParams& p, int n_resident, hipStream_t s) {
  constexpr int lds_dq = DqLds<DQK, DV, 1, false>::BYTES, lds_dkdv = DkdvLds<DQK, DV>::bytes();
  constexpr int lds = lds_dq > lds_dkdv ? lds_dq : lds_dkdv;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute((const void*)bwd_both4_kernel<DQK, DV>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  const int n_dkdv = p.n_tiles * p.Hkv * p.n_split, n_dq = p.n_q_tiles * p.Hq;
  hipLaunchKernelGGL((bwd_both4_kernel<DQK, DV>), dim3(n_dkdv + n_dq), dim3(kThreads), lds, s, p, n_dkdv, n_resident);
  return (int)hipGetLastError();
}

template <int DQK, int DV>
static int launch_bwd_t(const BwdParams& p, int grid_dq, int grid_dkdv, hipStream_t s, hipEvent_t* ev) {
  constexpr int lds_dq = DqLds<DQK, DV, 1, false>::BYTES, lds_dkdv = DkdvLds<DQK, DV>::bytes();
  const BwdItems items{PackShape{DQK, p.T, p.n_samples, p.Hq, p.Hkv}, p.n_tiles, p.n_q_tiles, p.n_split};
  const BwdLaunch how = bwd_launch(items, p.prof || p.prof_dq || ev[0] || ev[2]);
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)bwd_dq_kernel<DQK, DV>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_dq);
    if (e != hipSuccess) return (int)e;
    e = hipFuncSetAttribute((const void*)bwd_dkdv_kernel<DQK, DV>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds_dkdv);
    if (e != hipSuccess) return (int)e;
    attr_set = true;
  }
  {
    const bool small = (int64_t)p.T * p.Hq <= kPreSmall;
    const int hl = prepass_heads_log2(p.Hq), rows = (small ? 64 : 256) >> hl;
    const dim3 grid((unsigned)(((int64_t)p.T + rows - 1) / rows * ((p.Hq + (1 << hl) - 1) >> hl)));
    if (small) hipLaunchKernelGGL((bwd_prepass_kernel<DV, 64>), grid, dim3(kThreads), 0, s, p, hl);
    else hipLaunchKernelGGL((bwd_prepass_kernel<DV, 256>), grid, dim3(kThreads), 0, s, p, hl);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  if constexpr (DQK == DV) {
    if (how.one) {
      const int err = p.g % 2 == 0 ? launch_both<DQK, DV, true>(p, grid_dkdv, how.interleaved, s)
                                   : launch_both<DQK, DV, false>(p, grid_dkdv, how.interleaved, s);
      if (err) return err;
    }
  } else if (how.one) {
    const int err = launch_both4<DQK, DV>(p, grid_dkdv, s);
    if (err) return err;
  }
  if (grid_dkdv > 0) {
    if (ev[0] && hipEventRecord(ev[0], s) != hipSuccess) return (int)hipErrorInvalidValue;
    if constexpr (DQK == DV) {
      if (how.eight && !how.one) {
        const int err = launch_dkdv8<DQK, DV>(p, grid_dkdv, s);
        if (err) return err;
      }
    }
    if (!how.eight && !how.one)
      hipLaunchKernelGGL((bwd_dkdv_kernel<DQK, DV>), dim3(grid_dkdv), dim3(kThreads), lds_dkdv, s, p);
    e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    if (p.n_split > 1) {
      const int units = 128 * p.Hkv * ((DQK + DV) / 4);  // of a full tile; fewer than 8 kv heads here
      hipLaunchKernelGGL((bwd_reduce_parts_kernel<DQK, DV>), dim3(p.n_tiles, units / (kThreads * kReduceUnits)),
                         dim3(kThreads), 0, s, p);
      e = hipGetLastError();
      if (e != hipSuccess) return (int)e;
    }
    if (ev[1] && hipEventRecord(ev[1], s) != hipSuccess) return (int)hipErrorInvalidValue;
  }
  if (grid_dq > 0 && !how.one) {
    if (ev[2] && hipEventRecord(ev[2], s) != hipSuccess) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL((bwd_dq_kernel<DQK, DV>), dim3(grid_dq), dim3(kThreads), lds_dq, s, p);
    e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    if (ev[3] && hipEventRecord(ev[3], s) != hipSuccess) return (int)hipErrorInvalidValue;
  }
  return (int)e;
}

int launch_bwd(int d_qk, int d_v, const BwdParams& p, int grid_dq, int grid_dkdv, hipStream_t s,
               hipEvent_t* ev) {
  if (d_qk == 64 && d_v == 64) return launch_bwd_t<64, 64>(p, grid_dq, grid_dkdv, s, ev);
  if (d_qk == 128 && d_v == 128) return launch_bwd_t<128, 128>(p, grid_dq, grid_dkdv, s, ev);
  if (d_qk == 192 && d_v == 128) return launch_bwd_t<192, 128>(p, grid_dq, grid_dkdv, s, ev);
  return (int)hipErrorInvalidValue;
}

}  // namespace hbp
