// Block shapes of the sampler: column checkpoints, walkers per block and where
// its vectors are kept, chosen per launch from the sizes of the state.
#pragma once
#include "rtt_chain.hpp"
#include "rtt_host.hpp"

namespace rtt_host {

// Column checkpoints for a sweep launch: as many as CheckpointRule fits in
// LDS (half of it with more blocks of 16 walkers than compute units, at most
// 16), evenly spaced over the bonds a proposal can start its columns from,
// [lo, L), lo being passed in ck_first.
inline void chain_checkpoints(rttk::ChainArgs& a, int chi) {
  const int lo = a.ck_first, LW = (a.L + 63) / 64;
  a.n_ck = 0; a.ck_first = 0; a.ck_step = 1;
  if (a.mode != 1 || lo >= a.L || lo < 1) return;
  const CheckpointRule l0(chi, a.T, LW, a.nw, 0, a.N);
  int nmax = 0;
  if (l0.seq) {
    // (bond 256: the vectors are in global memory, which holds ck_cap of them)
    if (chi != 256) return;
    for (int n = std::min(16, a.ck_cap); n >= 1 && nmax == 0; --n)
      if (CheckpointRule(chi, a.T, LW, a.nw, n, a.N).total <= kLdsLimit) nmax = n;
  } else {
    if (chi > 64) return;
    const size_t budget = kLdsLimit / ((a.W + 15) / 16 > device_cus() ? 2 : 1);
    // the largest count that fits, preferring counts that keep the replica
    // bitmasks in LDS as they are without checkpoints
    for (int pass = 0; pass < 2 && nmax == 0; ++pass)
      for (int n = 16; n >= 1; --n) {
        const CheckpointRule ln(chi, a.T, LW, a.nw, n, a.N);
        if (ln.total <= budget && (pass == 1 || ln.rml == l0.rml)) { nmax = n; break; }
      }
  }
  if (nmax < 1) return;
  const int span = a.L - lo;
  const int step = (span + nmax - 1) / nmax;
  a.n_ck = (span + step - 1) / step;
  a.ck_first = lo;
  a.ck_step = step;
}

// LDS of a sampler block of this shape (persistent launches: no checkpoints)
template <class D, int CHI>
rttk::SampLayout samp_layout(const rttk::ChainArgs& a, int cg, int tw, bool ck_lds, bool p_lds) {
  const int sw = cg == 2 ? rttk::SampGeo<D, CHI, 2>::SW : tw == 2 ? rttk::SampGeo<D, CHI, 1, 2>::SW : rttk::SampGeo<D, CHI>::SW;
  return rttk::SampLayout(CHI, a.T, (a.L + 63) / 64, a.nw, cg, sw, tw, a.n_ck, ck_lds, p_lds);
}

// More walkers than one block of 16 on every compute unit: at the bonds that
// have both shapes a unit holds one block, and one round of 32 walkers is
// shorter than two of 16 (a sweep of 6000 walkers: BF16 128, 10x10 R=3, 23.8
// ms against 35.2; FP8 128, 8x8, 6.2 / 7.1; FP8 256, 9x9, two terms, 45.2 / 52.7;
// FP32 128, 6x6, 8.4 / 8.4), but longer than one of 16 (4096 walkers: 17.7, 3.8,
// 27.9 and 4.8 ms).
inline bool two_groups(int W) { return W > 16 * device_cus(); }

// The shape of a launch whose checkpoints are chosen: cg groups of 16 walkers
// per block, tw terms side by side, prefixes in global memory or in LDS.
// Bonds 128 and (FP8) 256 run two column groups per block from two_groups
// walkers on: each core fragment serves 32 walkers and is decoded once for
// them.  A block of 32 takes more
// LDS than the 16 walkers a state is accepted by: very long trains keep 16.
// Where one wave carries a whole vector, two terms of a combination advance
// side by side.
struct ChainShape {
  int cg, tw;
  bool p_global;
  int lds;
};
template <class D, int CHI>
ChainShape chain_shape(const rttk::ChainArgs& a) {
  constexpr bool kGlobal = CHI == 256 && std::is_same<D, rttk::DFP8>::value;
  ChainShape s{1, 1, false, 0};
  if constexpr (CHI == 128 || kGlobal) {
    s.lds = samp_layout<D, CHI>(a, 2, 1, !kGlobal, !kGlobal).total;
    if (two_groups(a.W) && s.lds <= (int)kLdsLimit) {
      s.cg = 2;
      s.p_global = kGlobal;
      return s;
    }
  }
  if (rttk::SampGeo<D, CHI, 1, 2>::SW == 1 && a.T > 1) s.tw = 2;
  s.lds = samp_layout<D, CHI>(a, 1, s.tw, !kGlobal, true).total;
  return s;
}

}  // namespace rtt_host
