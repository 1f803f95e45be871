// Flip-ratio passes of one core type, RTT_CORES = DF32, DBF16 or DFP8, for
// every padded bond.  Built once per core type.
#include <limits.h>

#include <type_traits>

#include "rtt_host.hpp"
#include "rtt_kernels.hpp"

namespace {

using namespace rtt_host;
using Cores = rttk::RTT_CORES;

constexpr int kDtype = rtt_host::kDtypeOf<Cores>;

template <class D, int CHI>
rtt_status launch_pass(const rttk::PassArgs& a, int T, hipStream_t s) {
  const bool wave = pass_wave(kDtype, CHI, a.nslot, (long)a.W * T);
  const int wpb = pass_walkers(CHI, wave);
  dim3 grid((a.W + wpb - 1) / wpb, T);
  if constexpr (rttk::pass_wave_bond<D, CHI>())
    if (wave) {
      hipLaunchKernelGGL((rttk::pass_wave_kernel<D, CHI>), grid, dim3(256), rtt_host::pass_wave_lds(kDtype, CHI), s, a);
      HIPX(hipGetLastError());
      return RTT_OK;
    }
  const size_t lds = pass_lds_bytes(CHI, a.nslot, a.nw, kDtype);
  auto kfn = rttk::pass_kernel<D, CHI>;
  HIPX(hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kfn, grid, dim3(256), lds, s, a);
  HIPX(hipGetLastError());
  return RTT_OK;
}

template <class D, int CHI>
rtt_status launch_batch(const BatchLaunch& b, bool prepare, hipStream_t s) {
  auto kfn = rttk::pass_persistent<D, CHI>;
  if (prepare) {  // before capture: allow the dynamic LDS size
    HIPX(hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b.pass_lds));
    return RTT_OK;
  }
  hipLaunchKernelGGL(kfn, dim3(b.grid_pass), dim3(256), b.pass_lds, s, b.d_pass, b.d_pass_items, b.n_pass, b.counter);
  HIPX(hipGetLastError());
  return RTT_OK;
}

rtt_status pass_any(int chi, const rttk::PassArgs& a, int T, hipStream_t s) {
  return by_bond<Cores>(chi, [&](auto c) { return launch_pass<Cores, decltype(c)::value>(a, T, s); });
}
rtt_status batch_any(int chi, const BatchLaunch& b, bool prepare, hipStream_t s) {
  return by_bond<Cores>(chi, [&](auto c) { return launch_batch<Cores, decltype(c)::value>(b, prepare, s); });
}

}  // namespace

#define RTT_CAT_(x, y) x##y
#define RTT_CAT(x, y) RTT_CAT_(x, y)
const rtt_host::PassLaunch* rtt_host::RTT_CAT(pass_, RTT_CORES)() {
  static const PassLaunch table = {pass_any, batch_any};
  return &table;
}
