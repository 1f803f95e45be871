// Sampler of one core type, RTT_CORES = DF32, DBF16 or DFP8, for every padded
// bond.  Built once per core type.
#include <limits.h>

#include <type_traits>

#include "rtt_shape.hpp"

namespace {

using namespace rtt_host;
using Cores = rttk::RTT_CORES;

template <class D, int CHI, int CG, int TW, bool CKP, bool CKG, bool PG>
rtt_status launch_chain_as(const rttk::ChainArgs& a, int lds, hipStream_t s) {
  if (lds > (int)kLdsLimit) return fail(RTT_E_UNSUPPORTED, "sampler: %d bytes of LDS needed", lds);
  auto kfn = rttk::chain_kernel<D, CHI, CG, TW, CKP, CKG, PG>;
  HIPX(hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
  hipLaunchKernelGGL(kfn, dim3((a.W + 16 * CG - 1) / (16 * CG)), dim3(2 * rttk::SampGeo<D, CHI, CG, TW>::SW * TW * 64),
                     lds, s, a);
  HIPX(hipGetLastError());
  return RTT_OK;
}

template <class D, int CHI>
rtt_status launch_chain(const rttk::ChainArgs& a0, hipStream_t s) {
  rttk::ChainArgs a = a0;
  chain_checkpoints(a, CHI);
  ChainShape sh = chain_shape<D, CHI>(a);
  if constexpr (CHI == 256 && std::is_same<D, rttk::DFP8>::value) {
    if (sh.cg == 2 && !a.pg && a.mode == 1) {  // no memory for the prefixes: blocks of 16
      sh.cg = 1;
      sh.lds = samp_layout<D, CHI>(a, 1, 1, false, true).total;
    }
    if (sh.cg == 2) return launch_chain_as<D, CHI, 2, 1, true, true, true>(a, sh.lds, s);
    return launch_chain_as<D, CHI, 1, 1, true, true, false>(a, sh.lds, s);
  } else if constexpr (CHI >= 128) {
    if constexpr (CHI == 128)
      if (sh.cg == 2) return launch_chain_as<D, CHI, 2, 1, false, false, false>(a, sh.lds, s);
    return launch_chain_as<D, CHI, 1, 1, false, false, false>(a, sh.lds, s);
  } else {
    if constexpr (rttk::SampGeo<D, CHI, 1, 2>::SW == 1)
      if (sh.tw == 2) return launch_chain_as<D, CHI, 1, 2, true, false, false>(a, sh.lds, s);
    return launch_chain_as<D, CHI, 1, 1, true, false, false>(a, sh.lds, s);
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
bool prefix_any(int chi, const rttk::ChainArgs& a0) {
  rttk::ChainArgs a = a0;
  chain_checkpoints(a, chi);
  bool global = false;
  (void)by_bond<Cores>(chi, [&](auto c) {
    global = chain_shape<Cores, decltype(c)::value>(a).p_global;
    return RTT_OK;
  });
  return global;
}

}  // namespace

#define RTT_CAT_(x, y) x##y
#define RTT_CAT(x, y) RTT_CAT_(x, y)
const rtt_host::ChainLaunch* rtt_host::RTT_CAT(chain_, RTT_CORES)() {
  static const ChainLaunch table = {chain_any, batch_any, batch_lds_any, prefix_any};
  return &table;
}
