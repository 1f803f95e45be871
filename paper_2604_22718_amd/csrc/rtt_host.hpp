// Host side shared by the translation units of librtt: errors, the on-chip
// memory rules, and the entry points through which rtt_lib.hip launches the
// kernels of a core type (rtt_pass.hip and rtt_chain.hip,
// built once per core type).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "../../include/rtt.h"
#include "rtt_kernels.hpp"

namespace rtt_host {

rtt_status fail(rtt_status st, const char* fmt, ...);

#define HIPX(call)                                                                             \
  do {                                                                                         \
    hipError_t e_ = (call);                                                                    \
    if (e_ != hipSuccess)                                                                      \
      return rtt_host::fail(e_ == hipErrorOutOfMemory ? RTT_E_OOM : RTT_E_HIP, "%s: %s (%s:%d)", \
                            #call, hipGetErrorString(e_), __FILE__, __LINE__);                 \
  } while (0)

constexpr size_t kLdsLimit = 160 * 1024;

inline int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

// Bytes that seven FP32 vectors per term (or, `seq`, one per term and five
// shared), nck column checkpoints with as many candidates, and a block's
// small state take: the rule by which states are accepted and by which the
// number of checkpoints follows.  Blocks of 16 walkers never need more
// (SampLayout), blocks of 32 can, and the checkpoints decide where the rows and columns of a proposal meet and
// with it the last bits of its amplitude, so the rule is part of what a
// seeded chain reproduces.
struct CheckpointRule {
  size_t total;
  bool seq, rml;
  CheckpointRule(int chi, int T, int LW, int nw, int nck, int n_spins) {
    const size_t nb = 16, bufb = nb * (chi + 4) * 4;
    seq = T * 7 * bufb + 4 * T * nb * 4 + T * nb * 12 + 8 + nb * (LW + nw) * 8 > 160 * 1024;
    const size_t vals = (seq ? T + 5 : (size_t)(7 + 2 * nck) * T) * bufb + 4 * T * nb * 4;
    const size_t pm = (vals + T * nb * 12 + 7) & ~(size_t)7;
    total = pm + nb * (LW + nw) * 8 + (size_t)2 * nck * T * nb * 4;
    const size_t rm = (total + 7) & ~(size_t)7;
    rml = rm + (size_t)n_spins * LW * 8 <= 160 * 1024;
    if (rml) total = rm + (size_t)n_spins * LW * 8;
  }
};

inline int rttk_wpw(int chi) { return chi >= 64 ? 4 : chi / 16; }

// the passes of rttk::pass_wide_form run the K-outer form (rows in place
// when so built, and at most kPassWideTiles row tiles per walker)
inline bool pass_wide(int dtype, int chi) {
  return PASS_W_ENABLE && ((dtype == RTT_FP8_E4M3 && (chi == 256 || (PASS_W_128 && chi == 128))) ||
                           (dtype == RTT_BF16 && PASS_W_128 && chi == 128));
}
inline int pass_max_slots(int dtype, int chi) { return pass_wide(dtype, chi) ? 16 * rttk::kPassWideTiles : 1 << 30; }

inline size_t pass_lds_bytes(int chi, int nslot, int nw, int dtype) {
  const int wpw = chi >= 64 ? 4 : chi / 16;
  const int wpb = 4 / wpw;
  const size_t rs = chi + 4;
  const int nb = (pass_wide(dtype, chi) && rttk::kPassWideInPlace) ? 1 : 2;  // row buffers
  return (size_t)wpb * (nb * nslot * rs * 4 + nb * nslot * 4 + nw * 8);
}

// Passes whose rows stay in the registers of one wave per walker, where a
// group's schedule has no more rows than that holds (up to 79 spins, or 159 in
// two groups; more take the rows-in-LDS form): at bond 32 for any number of
// walkers (8x8, BF16 evaluation: 16 walkers 160 -> 147 us, 4096 472 -> 328 us);
// at bond 64 from a pass per SIMD, where the rows-in-LDS form's four waves per
// walker queue for the chip (8x8: 1024 walkers 316 -> 250 us, 4096 941 -> 615
// us; below that a lone wave's chain of steps is the longer, 512 walkers 191
// against 241 us).  passes: walkers x terms x row groups of the launch.
inline bool pass_wave(int dtype, int chi, int nslot, long passes) {
  return dtype != RTT_F32 && chi <= 64 && nslot <= 16 * rttk::kPassWaveTiles &&
         (chi <= 32 || passes >= 4L * device_cus());
}
inline size_t pass_wave_lds(int dtype, int chi) { return rttk::pass_wave_lds(chi, dtype == RTT_FP8_E4M3 ? 1 : 2); }
// walkers per block of a pass
inline int pass_walkers(int chi, bool wave) { return wave ? 4 : 4 / rttk_wpw(chi); }

// Sampler tile of a class: 16 walkers per block, or 32 (two column groups
// sharing every core fragment) at bonds 32 and 128.  At 64 the second group
// spilled when vectors were in LDS (with vectors in registers it was not tried),
// and at 256 the prefixes of 32 do not fit in LDS (a single state keeps them in
// global memory).
constexpr bool batch_cg2(int chi) { return chi == 32 || chi == 128; }

// One class of a batch as its persistent kernels are launched
struct BatchLaunch {
  int cg, grid_chain, grid_pass;
  size_t chain_lds, pass_lds;
  const rttk::ChainArgs* d_chain;
  const rttk::PassArgs* d_pass;
  const int4 *d_chain_items, *d_pass_items;
  int n_chain, n_pass;
  int* counter;
  const uint64_t* sweep0;
};

// The kernels of one core type, by padded bond.  `batch` launches the
// persistent form of a class, or (prepare) allows its LDS size before capture.
struct PassLaunch {
  rtt_status (*run)(int chi, const rttk::PassArgs& a, int T, hipStream_t s);
  rtt_status (*batch)(int chi, const BatchLaunch& b, bool prepare, hipStream_t s);
};
struct ChainLaunch {
  rtt_status (*run)(int chi, const rttk::ChainArgs& a, hipStream_t s);
  rtt_status (*batch)(int chi, const BatchLaunch& b, bool prepare, hipStream_t s);
  // LDS of a persistent sampler block (one term at a time, no checkpoints)
  size_t (*batch_lds)(int chi, int T, int L, int nw, int cg);
  // whether a launch keeps its prefixes in global memory (pg), if given any
  bool (*global_prefix)(int chi, const rttk::ChainArgs& a);
};
const PassLaunch* pass_DF32();
const PassLaunch* pass_DBF16();
const PassLaunch* pass_DFP8();
const ChainLaunch* chain_DF32();
const ChainLaunch* chain_DBF16();
const ChainLaunch* chain_DFP8();

inline const PassLaunch* pass_launch(int dtype) {
  return dtype == RTT_F32 ? pass_DF32() : dtype == RTT_BF16 ? pass_DBF16() : pass_DFP8();
}
inline const ChainLaunch* chain_launch(int dtype) {
  return dtype == RTT_F32 ? chain_DF32() : dtype == RTT_BF16 ? chain_DBF16() : chain_DFP8();
}

template <class D>
constexpr int kDtypeOf = std::is_same<D, rttk::DFP8>::value    ? RTT_FP8_E4M3
                         : std::is_same<D, rttk::DBF16>::value ? RTT_BF16
                                                               : RTT_F32;

// f(bond) for the padded bonds this core type has kernels for
template <class Cores, class F>
rtt_status by_bond(int chi, F&& f) {
  using std::integral_constant;
  switch (chi) {
    case 16:
      if constexpr (Cores::kF32) return f(integral_constant<int, 16>{});
      break;
    case 32: return f(integral_constant<int, 32>{});
    case 64: return f(integral_constant<int, 64>{});
    case 128: return f(integral_constant<int, 128>{});
    case 256:
      if constexpr (!Cores::kF32) return f(integral_constant<int, 256>{});
      break;
  }
  return fail(RTT_E_UNSUPPORTED, "no kernel for dtype %d, padded bond %d", kDtypeOf<Cores>, chi);
}

}  // namespace rtt_host
