// Sampler of one core type, RTT_CORES = DF32, DBF16 or DFP8, for every padded
// bond.  Built once per core type.
#include <limits.h>

#include <type_traits>

#include "rtt_chain.hpp"
#include "rtt_host.hpp"

namespace {

using namespace rtt_host;
using Cores = rttk::RTT_CORES;

constexpr int kDtype = rtt_host::kDtypeOf<Cores>;

// Column checkpoints for a sweep launch: as many as CheckpointRule fits in
// LDS (half of it with more blocks of 16 walkers than compute units, at most
// 16), evenly spaced over the bonds a proposal can start its columns from,
// [lo, L), lo being passed in ck_first.
void chain_checkpoints(rttk::ChainArgs& a, int chi) {
  const int lo = a.ck_first, LW = (a.L + 63) / 64;
  a.n_ck = 0; a.ck_first = 0; a.ck_step = 1;
  if (a.mode != 1 || lo >= a.L || lo < 1) return;
  const CheckpointRule l0(chi, a.T, LW, a.nw, 0, a.N);
  int nmax = 0;
  if (l0.seq) {
    // (bond 256: the vectors are in global memory)
    if (chi != 256 || !a.ckg) return;
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
  const int sw = cg == 2 ? rttk::SampGeo<D, CHI, 2>::SW : rttk::SampGeo<D, CHI, 1>::SW;
  return rttk::SampLayout(CHI, a.T, (a.L + 63) / 64, a.nw, cg, sw, tw, a.n_ck, ck_lds, p_lds);
}

template <class D, int CHI, int CG, int TW, bool CKP, bool CKG, bool PG>
rtt_status launch_chain_as(const rttk::ChainArgs& a, hipStream_t s) {
  const rttk::SampLayout lay = samp_layout<D, CHI>(a, CG, TW, !CKG, !PG);
  if (lay.total > (int)kLdsLimit) return fail(RTT_E_UNSUPPORTED, "sampler: %d bytes of LDS needed", lay.total);
  auto kfn = rttk::chain_kernel<D, CHI, CG, TW, CKP, CKG, PG>;
  HIPX(hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, lay.total));
  hipLaunchKernelGGL(kfn, dim3((a.W + 16 * CG - 1) / (16 * CG)), dim3(2 * rttk::SampGeo<D, CHI, CG>::SW * TW * 64),
                     lay.total, s, a);
  HIPX(hipGetLastError());
  return RTT_OK;
}

// Bonds 128 and (FP8) 256 with enough walkers to give every CU a block of 32
// run two column groups per block: each core fragment serves 32 walkers and
// is decoded once for them (9x9, two FP8 terms, 8192 walkers: 80.6 ms a sweep
// with 16 walkers per block before, 48.8 with 32).  Up
// to bond 64, where one wave carries a whole vector, two terms of a
// combination advance side by side.
template <class D, int CHI>
rtt_status launch_chain(const rttk::ChainArgs& a0, hipStream_t s) {
  rttk::ChainArgs a = a0;
  chain_checkpoints(a, CHI);
  if constexpr (CHI == 256 && std::is_same<D, rttk::DFP8>::value) {
    if (two_groups(a.W) && (a.pg || a.mode == 0)) return launch_chain_as<D, CHI, 2, 1, true, true, true>(a, s);
    return launch_chain_as<D, CHI, 1, 1, true, true, false>(a, s);
  } else if constexpr (CHI >= 128) {
    if constexpr (CHI == 128)
      if (two_groups(a.W) && samp_layout<D, CHI>(a, 2, 1, true, true).total <= (int)kLdsLimit)
        return launch_chain_as<D, CHI, 2, 1, false, false, false>(a, s);
    return launch_chain_as<D, CHI, 1, 1, false, false, false>(a, s);
  } else {
    if constexpr (rttk::SampGeo<D, CHI>::SW == 1)
      if (a.T > 1) return launch_chain_as<D, CHI, 1, 2, true, false, false>(a, s);
    return launch_chain_as<D, CHI, 1, 1, true, false, false>(a, s);
  }
}

template <class D, int CHI>
rtt_status launch_batch(const BatchLaunch& b, bool prepare, hipStream_t s) {
  auto kfn = rttk::chain_persistent<D, CHI, 1>;
  int threads = 2 * rttk::SampGeo<D, CHI, 1>::SW * 64;
  if constexpr (batch_cg2(CHI))
    if (b.cg == 2) {
      kfn = rttk::chain_persistent<D, CHI, 2>;
      threads = 2 * rttk::SampGeo<D, CHI, 2>::SW * 64;
    }
  if (prepare) {  // before capture: allow the dynamic LDS size
    HIPX(hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b.chain_lds));
    return RTT_OK;
  }
  hipLaunchKernelGGL(kfn, dim3(b.grid_chain), dim3(threads), b.chain_lds, s, b.d_chain,
                     b.d_chain_items, b.n_chain, b.counter, b.sweep0);
  HIPX(hipGetLastError());
  return RTT_OK;
}

rtt_status chain_any(int chi, const rttk::ChainArgs& a, hipStream_t s) {
  return by_bond<Cores>(chi, [&](auto c) { return launch_chain<Cores, decltype(c)::value>(a, s); });
}
rtt_status batch_any(int chi, const BatchLaunch& b, bool prepare, hipStream_t s) {
  return by_bond<Cores>(chi, [&](auto c) { return launch_batch<Cores, decltype(c)::value>(b, prepare, s); });
}
size_t batch_lds_any(int chi, int T, int L, int nw, int cg) {
  rttk::ChainArgs a{};
  a.T = T; a.L = L; a.nw = nw;
  size_t bytes = (size_t)1 << 30;
  (void)by_bond<Cores>(chi, [&](auto c) {
    bytes = samp_layout<Cores, decltype(c)::value>(a, cg, 1, true, true).total;
    return RTT_OK;
  });
  return bytes;
}

}  // namespace

#define RTT_CAT_(x, y) x##y
#define RTT_CAT(x, y) RTT_CAT_(x, y)
const rtt_host::ChainLaunch* rtt_host::RTT_CAT(chain_, RTT_CORES)() {
  static const ChainLaunch table = {chain_any, batch_any, batch_lds_any};
  return &table;
}
