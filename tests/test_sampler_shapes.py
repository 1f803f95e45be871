"""Every state that rtt_create accepts has a sampler block that fits on chip,
whatever the number of walkers: the library's own shape rule is compiled into a
small host program and scanned over core types, bonds, terms, train lengths and
spin counts, up to where the acceptance rule ends."""
import json
import os
import subprocess

from paper_2604_22718_amd import build

PROGRAM = r"""
#include <cstdio>
#include "rtt_shape.hpp"
using namespace rtt_host;
rtt_status rtt_host::fail(rtt_status st, const char*, ...) { return st; }

struct Count { long accepted = 0, over = 0, two = 0, kept16 = 0; };

template <class D, int CHI>
void check(const rttk::ChainArgs& a0, bool seq, Count& n) {
  rttk::ChainArgs a = a0;
  constexpr bool global = CHI == 256 && std::is_same<D, rttk::DFP8>::value;
  a.ck_cap = global && seq && a.ck_first < a.L ? 8 : 0;
  chain_checkpoints(a, CHI);
  const ChainShape s = chain_shape<D, CHI>(a);
  const bool wide = (CHI == 128 || global) && two_groups(a.W);
  // the launch, the same without memory for prefixes, and a batch's block
  rttk::ChainArgs b = a;
  b.n_ck = 0;
  const int most = std::max({s.lds, samp_layout<D, CHI>(a, 1, s.tw, !global, true).total,
                             samp_layout<D, CHI>(b, 1, 1, true, true).total + 16});
  ++n.accepted;
  if (most > (int)kLdsLimit || s.lds <= 0 || (s.cg == 2) > wide || s.p_global != (global && s.cg == 2)) {
    if (n.over++ < 3)
      fprintf(stderr, "dtype %d bond %d T %d L %d N %d W %d: %d bytes\n", kDtypeOf<D>, CHI, a.T, a.L, a.N, a.W, most);
  }
  if (wide) ++(s.cg == 2 ? n.two : n.kept16);
}

template <class D>
void scan(Count& n) {
  for (int chi : {16, 32, 64, 128, 256})
    for (int T = 1; T <= 8; ++T)
      for (int N : {1, 64, 65, 100, 256, 500, 1000, 1024})
        for (int LW = 1; LW < 1280; LW += LW < 32 ? 1 : 2) {
          const int nw = (N + 63) / 64;
          const CheckpointRule rule(chi, T, LW, nw, 0, N);
          if (rule.total > kLdsLimit) break;
          for (int L : {64 * LW - 63, 64 * LW})
            for (int W : {1, 4097, 8191, 8192, 100000})
              for (int mode : {0, 1})
                for (int lo : {1, L / 2, L}) {
                  rttk::ChainArgs a{};
                  a.T = T; a.L = L; a.N = N; a.nw = nw; a.LW = LW; a.W = W; a.mode = mode; a.ck_first = lo;
                  (void)by_bond<D>(chi, [&](auto c) {
                    check<D, decltype(c)::value>(a, rule.seq, n);
                    return RTT_OK;
                  });
                }
        }
}

int main() {
  Count n;
  scan<rttk::DF32>(n);
  scan<rttk::DBF16>(n);
  scan<rttk::DFP8>(n);
  printf("{\"accepted\": %ld, \"over\": %ld, \"two\": %ld, \"kept16\": %ld}\n", n.accepted, n.over, n.two, n.kept16);
}
"""


def test_every_accepted_state_has_a_block_that_fits(tmp_path):
    src, exe = tmp_path / "shapes.hip", tmp_path / "shapes"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), "-Wno-unused-result", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300, check=True)
    n = json.loads(r.stdout)
    assert n["over"] == 0, r.stderr
    # both shapes occur, and so does the long train that keeps 16 walkers per block
    assert n["accepted"] > 100000 and n["two"] > 0 and n["kept16"] > 0, n
