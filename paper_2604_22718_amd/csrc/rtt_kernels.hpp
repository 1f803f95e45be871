// HIP kernels of the RTT Monte Carlo path (gfx950).
//
//  pass_kernel     one contraction pass of the flip-ratio schedule: the base
//                  environment vector plus one flipped vector per spin, all
//                  advanced core by core on the matrix cores (forward: row
//                  vectors from the left boundary to the cut bond; backward:
//                  column vectors from the right boundary to the cut).
#pragma once
#include <float.h>
#include <math.h>

#include <type_traits>

#include "rtt_device.hpp"
#include "rtt_tile.hpp"

namespace rttk {

constexpr int kMaxTerms = 8;
#ifndef PASS_PF_FP8
#define PASS_PF_FP8 2
#endif
// steps between power-of-two renormalisations: a row grows by at most chi
// per step, so 8 steps stay below 2^64 even at chi = 256 (FP32 range 2^128)
constexpr int kRenormEvery = 8;

template <int CHI>
struct Geo {
  static constexpr int WPW = CHI >= 64 ? 4 : CHI / 16;  // waves per walker / chain
  static constexpr int MT = CHI / (16 * WPW);           // 16-feature output tiles per wave
  static constexpr int KPL = CHI / 4;                   // input features per lane per row
  static constexpr int RS = CHI + 4;                    // LDS row stride (floats)
};

// ============================================================================
// pass kernel
// ============================================================================
// Schedule entry (int4): x = core position k, y = spin q read at k,
// z = active rows after this step, w = odd row (in | out << 16).  The odd row
// is the row of spin q: on the step where q first appears it is spawned from
// the base row (in = 0), otherwise it is q's own row (in = out).  It uses
// slice 1 - s_q; every other active row uses slice s_q.
struct PassArgs {
  const void* cores;        // [T][L][2][CHI*CHI], fragment layout of this direction
  const int32_t* core_exp;  // [T][L] power-of-two scale exponents, or null
  const int4* sched;        // schedules of all row groups, concatenated
  const int2* gsteps;       // [ng] (first entry, number of entries) of each group
  int ng;                   // row groups: spins are split so a group's rows fit on chip
  int nslot;                // rows per walker and group, multiple of 16
  int L, nw, W;
  const uint64_t* spins;    // [W][nw]
  float* out_vec;           // [T][ng][W][nslot][CHI]
  int32_t* out_exp;         // [T][ng][W][nslot]
  int wave;                 // batched passes: items are for the wave-resident form
};

// ----------------------------------------------------------------------------
// Flip-ratio pass with the K loop outermost (FP8 cores at bond 256, BF16 and
// FP8 cores at bond 128).  One walker per block; wave wv owns output
// features [wv chi / 4, (wv + 1) chi / 4), MT = chi / 64 tiles of 16.  For
// each 32-wide K chunk a lane's 8 core values of every tile are taken from
// its fragment word once (FP8 codes decoded to BF16), each active row tile's
// activations for that chunk are read from LDS once and multiplied into the
// MT tiles' accumulators, which stay live for the whole step.  Every
// accumulator sees the matrix-op sequence of pass_body (chunk by chunk, hi
// part then lo part), so the results are the same bits.
// With PASS_W_INPL rows are updated in place: the step's outputs wait in
// registers until every wave has read its inputs, so a walker's rows take
// half the LDS and twice as many fit (fewer row groups, fewer core reads).
// Tuning on the 16x16 four-term workload (local energies, 16384 walkers):
// the double-buffered item form 2.75 s; K outermost, two buffers 2.59 s; in
// place with 6 row tiles 2.22 s; with 9 (two row groups instead of three)
// and the two-slot ring below 2.06 s; with each step compiled for its exact
// row-tile count (no per-tile branches) 1.61 s, and for whether it
// renormalises (no scaling on the other steps) 1.55 s.  A four-slot ring
// spills.
#ifndef PASS_W_NTM  // row tiles a group may hold
#define PASS_W_NTM 9
#endif
#ifndef PASS_W_INPL
#define PASS_W_INPL 1
#endif
#ifndef PASS_W_ENABLE  // 0: every pass runs pass_body's item form
#define PASS_W_ENABLE 1
#endif
#ifndef PASS_W_RING  // fragment ring slots: 4 = one step ahead, 2 = half a step
#define PASS_W_RING 2
#endif
constexpr int kPassWideTiles = PASS_W_NTM;        // row tiles a step may hold
constexpr bool kPassWideInPlace = PASS_W_INPL != 0;

// PASS_W_128 also runs FP8 and BF16 at bond 128 in this form (bit-identical
// there), compiled for two waves per SIMD (pass_min_blocks): 10x10 bond-128
// BF16 local energies 18.7 -> 16.7 ms against the item form; left free to
// use one wave per SIMD it was slower (30.2 ms).  BF16 at bond 256 spills
// in this form.
#ifndef PASS_W_128
#define PASS_W_128 1
#endif
template <class D, int CHI>
constexpr bool pass_wide_form() {
  return PASS_W_ENABLE && ((std::is_same<D, DFP8>::value && (CHI == 256 || (PASS_W_128 && CHI == 128))) ||
                           (std::is_same<D, DBF16>::value && PASS_W_128 && CHI == 128));
}

// blocks per CU the pass kernels are compiled for (a register budget): two
// for the bond-128 K-outer form, whose registers would otherwise grow past
// what two waves per SIMD allow
template <class D, int CHI>
constexpr int pass_min_blocks() { return (pass_wide_form<D, CHI>() && CHI == 128) ? 2 : 1; }

template <class D, int CHI>
__device__ __forceinline__ void pass_body_wide(const PassArgs& a, int bx, int ty) {
  constexpr bool F8 = std::is_same<D, DFP8>::value;
  constexpr int KPL = CHI / 4, MT = CHI / 64, RS = CHI + 4, NTM = kPassWideTiles;
  constexpr int NCH = KPL / 8;     // 32-wide K chunks per step
  constexpr int CPW = F8 ? 2 : 1;  // K chunks per 16-byte fragment word (FP8: 16 codes)
  constexpr int NWD = NCH / CPW;   // fragment words per lane and tile
  static_assert(NTM >= 1 && NTM <= 9, "the step dispatch covers 1 to 9 row tiles");
  constexpr bool INPL = kPassWideInPlace;
  constexpr int NB = INPL ? 1 : 2;  // row buffers
  using A = Act<D, CHI>;
  using E = typename D::elem;
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int g = lane >> 4, m = lane & 15;
  const int w = bx < a.W ? bx : a.W - 1;
  const int nslot = a.nslot;
  const int bufsz = nslot * RS;
  float* cur = lds;
  float* nxt = INPL ? lds : lds + bufsz;
  int* exc = reinterpret_cast<int*>(lds + NB * bufsz);
  int* exn = INPL ? exc : exc + nslot;
  uint64_t* spw = reinterpret_cast<uint64_t*>(lds + NB * bufsz + NB * nslot);
  for (int i = threadIdx.x; i < NB * bufsz; i += 256) cur[i] = 0.f;
  for (int i = threadIdx.x; i < NB * nslot; i += 256) exc[i] = 0;
  for (int i = threadIdx.x; i < a.nw; i += 256) spw[i] = a.spins[(size_t)w * a.nw + i];
  __syncthreads();
  if (threadIdx.x == 0) A::set_unit(cur);  // boundary vector e_0 in the base slot
  __syncthreads();

  const int term = ty / a.ng, grp = ty % a.ng;
  const E* cores = static_cast<const E*>(a.cores) + (size_t)term * a.L * 2 * CHI * CHI;
  const int* cexp_p = a.core_exp ? a.core_exp + (size_t)term * a.L : nullptr;
  const int2 gs = a.gsteps[grp];
  const int4* sched = a.sched + gs.x;
  const int n = gs.y;

  // Ring of fragment words: a slot holds one 16-byte word j of each lane's
  // fragment (elements 16j .. 16j + 15 for FP8 codes, 8j .. 8j + 7 for BF16)
  // of this wave's MT tiles, of the walker's slice (Rm) and, on steps with an
  // odd row, of the other slice (Ro).  A step streams its NWD words through
  // the RING slots; a slot is refilled with the word RING places further on
  // (in this step or the next) as soon as its K chunks are decoded, so every
  // load has RING / NWD of a step to arrive.
  constexpr int RING = PASS_W_RING < NWD ? PASS_W_RING : NWD;
  uint4 Rm[RING][MT], Ro[RING][MT];
  constexpr int TILE16 = 64 * KPL * (int)sizeof(E) / 16;  // 16-byte words per fragment tile
  // load word j of a step's fragments into ring slot j % RING
  auto issue = [&](int j, const int4& st, int bit) {
    const int sl = j % RING;
    const uint4* bm = reinterpret_cast<const uint4*>(cores + ((size_t)st.x * 2 + bit) * (CHI * CHI)) +
                      (size_t)wv * MT * TILE16;
#pragma unroll
    for (int q = 0; q < MT; ++q) Rm[sl][q] = bm[q * TILE16 + 64 * j + lane];
    if (st.w >= 0) {
      const uint4* bo = reinterpret_cast<const uint4*>(cores + ((size_t)st.x * 2 + (bit ^ 1)) * (CHI * CHI)) +
                        (size_t)wv * MT * TILE16;
#pragma unroll
      for (int q = 0; q < MT; ++q) Ro[sl][q] = bo[q * TILE16 + 64 * j + lane];
    }
  };
  // the A operand of K chunk c from its fragment word: FP8 codes 8c .. 8c + 7
  // (half h = c % 2 of the word) decoded to BF16, or the word's 8 BF16 values
  auto dec = [](const uint4& v, int h) -> bf16x8 {
    if constexpr (F8) {
      const uint32_t w0 = h ? v.z : v.x, w1 = h ? v.w : v.y;
      const auto p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, kFp8Scale, false);
      const auto p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, kFp8Scale, true);
      const auto p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, kFp8Scale, false);
      const auto p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, kFp8Scale, true);
      return bf16x8{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
    } else {
      return __builtin_bit_cast(bf16x8, v);
    }
  };

  if (n > 0) {
    const int4 st0 = sched[0];
    const int bit0 = spin_bit(spw, st0.y);
#pragma unroll
    for (int j = 0; j < RING; ++j) issue(j, st0, bit0);
  }
  for (int s = 0; s < n; ++s) {
    const int4 st = sched[s];
    const int k = st.x, nact = st.z, odd = st.w;
    const int oin = odd >= 0 ? (odd & 0xffff) : -1, oout = odd >> 16;
    const int ot = odd >= 0 ? (oin >> 4) : -1;  // row tile of the odd row's input
    const int ntile = (nact + 15) >> 4;
    // renormalise every kRenormEvery steps (a row grows by at most chi per step)
    const bool rn = (s % kRenormEvery) == 0;
    const int4 stn = sched[min(s + 1, n - 1)];
    const int bitc = spin_bit(spw, st.y), bitn = spin_bit(spw, stn.y);
    const int cexp = cexp_p ? cexp_p[k] : 0;
    const float* orow = cur + (16 * (ot < 0 ? 0 : ot) + m) * RS;  // the odd row's input tile
    // One step over exactly NT row tiles (dispatched below on the step's
    // tile count): no branch per tile, so the compiler is free to issue a
    // chunk's reads ahead of the matrix ops, and no accumulator of an idle
    // tile is carried through the K loop.
    auto step = [&](auto ntc, auto rnc) {
      constexpr int NT = decltype(ntc)::value;
      constexpr bool RN = decltype(rnc)::value;  // a renormalisation step
      f4 acc[NT][MT], oacc[MT];
#pragma unroll
      for (int r = 0; r < NT; ++r) {
#pragma unroll
        for (int q = 0; q < MT; ++q) acc[r][q] = f4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int q = 0; q < MT; ++q) oacc[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int j = c / CPW, h = c % CPW, sl = j % RING;
        bf16x8 Am[MT];
#pragma unroll
        for (int q = 0; q < MT; ++q) Am[q] = dec(Rm[sl][q], h);
        // the odd row: the other slice applied to its input row (the same
        // LDS values its tile reads above)
        if (ot >= 0) {
          bf16x8 Ao[MT];
#pragma unroll
          for (int q = 0; q < MT; ++q) Ao[q] = dec(Ro[sl][q], h);
          const uint16_t* hp = A::hi(orow) + g * KPL + 8 * c;
          const bf16x8 bh = *reinterpret_cast<const bf16x8*>(hp);
          const bf16x8 bl = *reinterpret_cast<const bf16x8*>(hp + CHI);
#pragma unroll
          for (int q = 0; q < MT; ++q) {
            oacc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ao[q], bh, oacc[q], 0, 0, 0);
            oacc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ao[q], bl, oacc[q], 0, 0, 0);
          }
        }
        // the slot is free: refill it with the word RING places further on
        if (h == CPW - 1) {
          if (j + RING < NWD) issue(j + RING, st, bitc);
          else issue(j + RING - NWD, stn, bitn);
        }
#pragma unroll
        for (int r = 0; r < NT; ++r) {
          const uint16_t* hp = A::hi(cur + (16 * r + m) * RS) + g * KPL + 8 * c;
          const bf16x8 bh = *reinterpret_cast<const bf16x8*>(hp);
          const bf16x8 bl = *reinterpret_cast<const bf16x8*>(hp + CHI);
#pragma unroll
          for (int q = 0; q < MT; ++q) {
            acc[r][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Am[q], bh, acc[r][q], 0, 0, 0);
            acc[r][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Am[q], bl, acc[r][q], 0, 0, 0);
          }
        }
      }
      // per-row exponents on renormalisation steps, from a second read of
      // the rows' hi parts exactly as in pass_body (a running maximum carried
      // over the K chunks instead gave wrong values in row tiles after the
      // first; its cause was not identified, so that form is not used)
      int e[NT];
      int oe = 0;
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        e[r] = 0;
        if constexpr (RN) {
          DBF16::BOp<KPL> bo;
          A::template load_b<KPL>(cur + (16 * r + m) * RS, g, bo);
          e[r] = A::template row_exp<KPL>(bo);
        }
      }
      if (RN && ot >= 0) {  // the exponent of the odd row's input row
        DBF16::BOp<KPL> bo;
        A::template load_b<KPL>(orow, g, bo);
        oe = A::template row_exp<KPL>(bo);
      }
      // exponents are read and written by wave 0 alone (program order); rows
      // are read by every wave, so in place they wait for the barrier
      int eold[NT];
      int eoin = 0;
      if (wv == 0) {
#pragma unroll
        for (int r = 0; r < NT; ++r) eold[r] = exc[16 * r + m];
        if (oin >= 0) eoin = exc[oin];
      }
      if (INPL) lds_barrier();
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        const float sc = __builtin_amdgcn_ldexpf(1.f, -e[r]);  // exact power of two
#pragma unroll
        for (int q = 0; q < MT; ++q) {
          f4 v = acc[r][q];
          if constexpr (RN) {  // the scale is 1 on other steps
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= sc;
          }
          A::store4(nxt + (16 * r + m) * RS, g * KPL + 4 * (wv * MT + q), v);
        }
        if (wv == 0 && g == 0) exn[16 * r + m] = eold[r] + e[r] + cexp;
      }
      if (oin >= 0) {  // lanes of column oin % 16 hold the odd row's outputs
        if (m == (oin & 15)) {
          const float sc = __builtin_amdgcn_ldexpf(1.f, -oe);
#pragma unroll
          for (int q = 0; q < MT; ++q) {
            f4 v = oacc[q];
            if constexpr (RN) {
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] *= sc;
            }
            A::store4(nxt + oout * RS, g * KPL + 4 * (wv * MT + q), v);
          }
        }
        if (wv == 0 && lane == (oin & 15)) exn[oout] = eoin + oe + cexp;
      }
    };
    // dispatched on the tile count and, as a second template parameter, on
    // whether the step renormalises (the other steps then carry no scaling)
    auto dispatch = [&](auto rnc) {
      switch (ntile) {
#define PASS_W_CASE(x)                                                     \
  case x:                                                                 \
    if constexpr (x <= NTM) step(std::integral_constant<int, x>{}, rnc);   \
    break;
        PASS_W_CASE(1) PASS_W_CASE(2) PASS_W_CASE(3) PASS_W_CASE(4) PASS_W_CASE(5)
        PASS_W_CASE(6) PASS_W_CASE(7) PASS_W_CASE(8) PASS_W_CASE(9)
#undef PASS_W_CASE
        default: break;  // the host keeps every group within NTM tiles
      }
    };
    if (rn) dispatch(std::true_type{});
    else dispatch(std::false_type{});
    lds_barrier();
    if (!INPL) {
      float* tp = cur; cur = nxt; nxt = tp;
      int* te = exc; exc = exn; exn = te;
    }
  }
  __syncthreads();

  if (bx < a.W) {
    float* ov = a.out_vec + (((size_t)ty * a.W + w) * nslot) * CHI;
    for (int i = threadIdx.x; i < nslot * CHI; i += 256) ov[i] = A::get(cur + (i / CHI) * RS, i % CHI);
    int32_t* oe_out = a.out_exp + ((size_t)ty * a.W + w) * nslot;
    for (int i = threadIdx.x; i < nslot; i += 256) oe_out[i] = exc[i];
  }
}

// ----------------------------------------------------------------------------
// Wave-resident flip-ratio pass (BF16 and FP8 cores up to bond 64): one wave
// per walker, every row in its registers from the boundary to the cut.  Every
// walker needs one slice of a site for its rows and, where the site's spin is
// of its group, the other for the odd row, so a block stages both for its four
// walkers, a site ahead, in two halves of LDS: one barrier per step, and a
// quarter of the slice traffic.  A row tile is multiplied chunk by chunk, hi
// part then lo part, as in pass_body (the results are the same bits), split
// and kept; the odd row is the column of its tile's product with the other
// slice, moved to its slot.
// Bound by issue: 16 matrix ops and 64 vector ops (split, selection) per row
// tile at bond 64, one more tile per step for the odd row.  8x8 BF16 bond 64,
// 4096 walkers, one pass: 446 us with the rows in LDS and four waves per
// walker, 280 us here (matrix ops alone 103 us).  With slices in registers
// instead of LDS the rows spilled (350 us), and at one wave per SIMD vector
// and matrix ops do not overlap (390 us).
// Up to kPassWaveTiles row tiles: five take 252 registers at bond 64, where
// two waves per SIMD have 256 each (at bond 32, 132: more were not tried).
constexpr int kPassWaveTiles = 5;
template <class D, int CHI>
constexpr bool pass_wave_bond() { return !D::kF32 && CHI <= 64; }
constexpr size_t pass_wave_lds(int chi, int elem_bytes) { return (size_t)4 * chi * chi * elem_bytes; }

template <int A, int B, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    static_for<A + 1, B>(f);
  }
}

template <class D, int CHI, int NTM>
__device__ __forceinline__ void pass_body_wave(const PassArgs& a, int bx, int ty) {
  using E = typename D::elem;
  using Op = TileOp<D, CHI>;
  using Fr = Frag<E, CHI / 4>;
  constexpr int NV = CHI / 16, KPL = CHI / 4, NCH = CHI / 32;
  constexpr int SLICE = CHI * CHI * (int)sizeof(E), TILE = 64 * KPL * (int)sizeof(E);
  constexpr int NS = (2 * SLICE + 4095) / 4096;  // 16-byte words of a site that a thread stages
  extern __shared__ __align__(16) float lds[];
  char* buf = reinterpret_cast<char*>(lds);  // [2][slice of bit 0, slice of bit 1]
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15;
  const int w_raw = bx * 4 + __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = min(w_raw, a.W - 1), term = ty / a.ng, grp = ty % a.ng;
  const char* cores = static_cast<const char*>(a.cores) + (size_t)term * a.L * 2 * SLICE;
  const int4* sched = a.sched + uniform_load(&a.gsteps[grp].x, 0);
  const int n = uniform_load(&a.gsteps[grp].y, 0);
  const uint64_t* spins = a.spins + (size_t)w * a.nw;
  u32x4 r[NTM][NV];
  int ex[NTM];
#pragma unroll
  for (int t = 0; t < NTM; ++t) {
    ex[t] = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) r[t][v] = u32x4{0, 0, 0, 0};
  }
  r[0][0][0] = lane == 0 ? Op::kUnit : 0u;  // boundary vector e_0 in the base slot
  // A step's entry is read three steps ahead and the walker's spin two; both
  // slices of the next site are on their way to LDS during a whole step.
  struct Step { int k, q, nact, odd, bit, cexp; };
  auto entry = [&](int s, Step& st) {
    const int* e = &sched[min(s, n - 1)].x;
    st.k = uniform_load(e, 0);
    st.q = uniform_load(e, 1);
    st.nact = uniform_load(e, 2);
    st.odd = uniform_load(e, 3);
  };
  auto spin = [&](Step& st) {
    st.bit = (int)((uniform_load(spins, st.q >> 6) >> (st.q & 63)) & 1ull);
    st.cexp = a.core_exp ? uniform_load(a.core_exp, (long long)term * a.L + st.k) : 0;
  };
  u32x4 stage[NS];
  auto fetch = [&](int k) {
    typedef const __attribute__((address_space(1))) u32x4* gvec;
    const gvec p = (gvec)(cores + (size_t)k * 2 * SLICE);
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if (16 * (256 * i + tid) < 2 * SLICE) stage[i] = p[256 * i + tid];
  };
  auto put = [&](int half) {
    u32x4* p = reinterpret_cast<u32x4*>(buf + half * 2 * SLICE);
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if (16 * (256 * i + tid) < 2 * SLICE) p[256 * i + tid] = stage[i];
  };
  auto read = [&](Fr& f, const char* p) {
    if constexpr (Fr::NW % 4 == 0) {
#pragma unroll
      for (int i = 0; i < Fr::NW / 4; ++i) {
        const u32x4 v = reinterpret_cast<const u32x4*>(p)[64 * i + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) f.w[4 * i + j] = v[j];
      }
    } else {
      const uint2 v = reinterpret_cast<const uint2*>(p)[lane];
      f.w[0] = v.x;
      f.w[1] = v.y;
    }
  };
  // output tile t of the vectors in times a slice, renormalised by sc, as words
  auto tile = [&](auto rnc, const Fr& f, const u32x4(&in)[NV], float sc, u32x4(&out)[NV], int t) {
    constexpr bool RN = decltype(rnc)::value;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      typename Op::Operand x;
#pragma unroll
      for (int q = 0; q < Op::kPieces; ++q) Op::decode(f, c, q, x);
#pragma unroll
      for (int h = 0; h < 2; ++h) acc = Op::op(x, in, c, h, acc);
    }
    typename Op::Post ps;
#pragma unroll
    for (int st = 0; st < Op::kStages; ++st) Op::template post<RN, NV>(st, ps, false, acc, acc, sc, out, t);
  };
  Step cur = {0, 0, 0, -1, 0, 0}, nxt = cur, n2 = cur;
  if (n > 0) {
    entry(0, cur);
    entry(1, nxt);
    entry(2, n2);
    spin(cur);
    spin(nxt);
    fetch(cur.k);
    put(0);
    lds_barrier();
  }
  auto step = [&](auto ntc, auto rnc, int half) {
    constexpr int NT = decltype(ntc)::value;
    constexpr bool RN = decltype(rnc)::value;
    const int oin = cur.odd >= 0 ? (cur.odd & 0xffff) : -1, oout = cur.odd >> 16;
    const char* own = buf + (half * 2 + cur.bit) * SLICE;
    const char* other = buf + (half * 2 + (cur.bit ^ 1)) * SLICE;
    // scale factor of a tile's product and its columns' exponents after the step
    auto rescale = [&](const u32x4(&x)[NV], int& e) {
      float sc = 1.f;
      if constexpr (RN) {
        const int me = Op::row_exp(x);
        sc = __builtin_amdgcn_ldexpf(1.f, -me);  // exact power of two
        e += me;
      }
      e += cur.cexp;
      return sc;
    };
    fetch(nxt.k);
    hold_loads();
    u32x4 ow[NV];
    int oe = ex[0];
#pragma unroll
    for (int v = 0; v < NV; ++v) ow[v] = r[0][v];
    if (oin >= 0) {
      u32x4 x[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) x[v] = r[0][v];
#pragma unroll
      for (int t = 1; t < NT; ++t)
        if (t == (oin >> 4)) {
          oe = ex[t];
#pragma unroll
          for (int v = 0; v < NV; ++v) x[v] = r[t][v];
        }
      const float sc = rescale(x, oe);
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        Fr f;
        read(f, other + t * TILE);
        tile(rnc, f, x, sc, ow, t);
      }
      if (oin == 0 && oout != 0) {  // spawned from the base row: column 0 to every column
        oe = __builtin_amdgcn_update_dpp(0, oe, 0x150, 0xf, 0xf, true);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            ow[v][i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ow[v][i], 0x150, 0xf, 0xf, true);
      }
    }
    Fr F[NV];
#pragma unroll
    for (int t = 0; t < NV; ++t) read(F[t], own + t * TILE);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float sc = rescale(r[t], ex[t]);
      u32x4 o[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) tile(rnc, F[v], r[t], sc, o, v);
#pragma unroll
      for (int v = 0; v < NV; ++v) r[t][v] = o[v];
    }
    if (oin >= 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bool mine = 16 * t + m == oout;
        ex[t] = mine ? oe : ex[t];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int i = 0; i < 4; ++i) r[t][v][i] = mine ? ow[v][i] : r[t][v][i];
      }
    }
    put(half ^ 1);
    lds_barrier();
  };
  // as many tiles as a step has rows for (their number only grows)
  int s = 0;
  static_for<1, NTM + 1>([&](auto ntc) {
    constexpr int NT = decltype(ntc)::value;
    while (s < n && (NT == NTM || cur.nact <= 16 * NT)) {
      Step n3 = n2;
      entry(s + 3, n3);
      spin(n2);
      if (s % kRenormEvery == 0) step(ntc, std::true_type{}, s & 1);
      else step(ntc, std::false_type{}, s & 1);
      cur = nxt;
      nxt = n2;
      n2 = n3;
      ++s;
    }
  });
  if (w_raw >= a.W) return;  // no barrier below
  const int g = lane >> 4;
  float* ov = a.out_vec + ((size_t)ty * a.W + w) * a.nslot * CHI;
  int32_t* oe_out = a.out_exp + ((size_t)ty * a.W + w) * a.nslot;
#pragma unroll
  for (int t = 0; t < NTM; ++t) {
    if (16 * t >= a.nslot) break;
    float* d = ov + (size_t)(16 * t + m) * CHI + g * KPL;
#pragma unroll
    for (int c = 0; c < NV / 2; ++c)
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // elements 8 c + 4 q .. + 3
        const uint32_t h0 = r[t][2 * c][2 * q], h1 = r[t][2 * c][2 * q + 1];
        const uint32_t l0 = r[t][2 * c + 1][2 * q], l1 = r[t][2 * c + 1][2 * q + 1];
        *reinterpret_cast<float4*>(d + 8 * c + 4 * q) = make_float4(
            __uint_as_float(h0 << 16) + __uint_as_float(l0 << 16),
            __uint_as_float(h0 & 0xffff0000u) + __uint_as_float(l0 & 0xffff0000u),
            __uint_as_float(h1 << 16) + __uint_as_float(l1 << 16),
            __uint_as_float(h1 & 0xffff0000u) + __uint_as_float(l1 & 0xffff0000u));
      }
    if (g == 0) oe_out[16 * t + m] = ex[t];
  }
}

// the body for the schedule's row tiles
template <class D, int CHI>
__device__ __forceinline__ void pass_wave_any(const PassArgs& a, int bx, int ty) {
  switch (a.nslot / 16) {
    case 1: pass_body_wave<D, CHI, 1>(a, bx, ty); break;
    case 2: pass_body_wave<D, CHI, 2>(a, bx, ty); break;
    case 3: pass_body_wave<D, CHI, 3>(a, bx, ty); break;
    case 4: pass_body_wave<D, CHI, 4>(a, bx, ty); break;
    default: pass_body_wave<D, CHI, 5>(a, bx, ty); break;
  }
}

template <class D, int CHI>
__global__ void __launch_bounds__(256, 2) pass_wave_kernel(PassArgs a) {
  pass_wave_any<D, CHI>(a, blockIdx.x, blockIdx.y);
}

template <class D, int CHI>
__device__ __forceinline__ void pass_body(const PassArgs& a, int bx, int ty) {
  if constexpr (pass_wide_form<D, CHI>()) {
    pass_body_wide<D, CHI>(a, bx, ty);
    return;
  }
  using E = typename D::elem;
  using G = Geo<CHI>;
  constexpr int WPW = G::WPW, MT = G::MT, KPL = G::KPL, RS = G::RS;
  constexpr int WPB = 4 / WPW;
  extern __shared__ __align__(16) float lds[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ws = wave / WPW, wv = wave % WPW;
  const int g = lane >> 4, m = lane & 15;
  const int w_raw = bx * WPB + ws;
  const int w = w_raw < a.W ? w_raw : a.W - 1;
  const int nslot = a.nslot;
  const int bufsz = nslot * RS;
  float* cur = lds + ws * (2 * bufsz);
  float* nxt = cur + bufsz;
  int* exc = reinterpret_cast<int*>(lds + WPB * 2 * bufsz) + ws * (2 * nslot);
  int* exn = exc + nslot;
  uint64_t* spw = reinterpret_cast<uint64_t*>(lds + WPB * 2 * bufsz + WPB * 2 * nslot) + ws * a.nw;

  const int tid_w = wv * 64 + lane;
  constexpr int NT_W = WPW * 64;
  for (int i = tid_w; i < 2 * bufsz; i += NT_W) cur[i] = 0.f;
  for (int i = tid_w; i < 2 * nslot; i += NT_W) exc[i] = 0;
  for (int i = tid_w; i < a.nw; i += NT_W) spw[i] = a.spins[(size_t)w * a.nw + i];
  __syncthreads();
  using A = Act<D, CHI>;
  if (tid_w == 0) A::set_unit(cur);  // boundary vector e_0 in the base slot
  __syncthreads();

  const int term = ty / a.ng, grp = ty % a.ng;
  const E* cores = static_cast<const E*>(a.cores) + (size_t)term * a.L * 2 * CHI * CHI;
  const int* cexp_p = a.core_exp ? a.core_exp + (size_t)term * a.L : nullptr;
  const int2 gs = a.gsteps[grp];
  const int4* sched = a.sched + gs.x;

  // Work items = (schedule step, group of MTI output tiles of this wave).
  // When the fragments of all MT tiles fit in registers (MTI = MT) a row
  // tile's activations are read once per step and used for every tile;
  // otherwise (bond 256) once per half of the tiles.  The core fragments of item i+1
  // are loaded while item i computes.  Rows are stored in the matrix-op
  // form (Act), and renormalisation scales the products, not the inputs.
  // (FP8 fragments are sized as BF16 ones here: the codes are decoded to
  // BF16 operands next to the matrix ops, which needs the room)
  constexpr int FRAG_DW = MT * 2 * KPL * (sizeof(E) < 2 ? 2 : (int)sizeof(E)) / 4;
  constexpr int MTI = FRAG_DW <= 128 ? MT : (MT % 2 == 0 && FRAG_DW <= 256 ? MT / 2 : 1);
  constexpr int NIS = MT / MTI;  // items per step
  constexpr bool ODD_MFMA = !D::kF32;
  struct Frags { Frag<E, KPL> m[MTI], o[MTI]; };
  // FP8 fragments stay codes while their loads are in flight and are decoded
  // to BF16 once per item, since every row tile of the step uses them; the
  // matrix ops then run as for BF16 cores
  constexpr bool kDec = std::is_same<D, DFP8>::value;
  using DR = typename std::conditional<kDec, DBF16, D>::type;
  using ER = typename DR::elem;
  const int n_items = gs.y * NIS;
  // The other slice is read only on steps with an odd row (one step in ng
  // when the spins are dealt over ng groups); elsewhere F.o keeps whatever
  // it held and is not used.
  auto load = [&](Frags& F, int item) {
    const int s = item / NIS, ig = item % NIS;
    const int4 st = sched[s];
    const int bit = spin_bit(spw, st.y);
#pragma unroll
    for (int q = 0; q < MTI; ++q) {
      const size_t tile = (size_t)(wv * MT + ig * MTI + q) * 64 * KPL;
      load_frag<E, KPL>(F.m[q], cores + ((size_t)st.x * 2 + bit) * (CHI * CHI) + tile, lane);
    }
    if (st.w >= 0) {
#pragma unroll
      for (int q = 0; q < MTI; ++q) {
        const size_t tile = (size_t)(wv * MT + ig * MTI + q) * 64 * KPL;
        load_frag<E, KPL>(F.o[q], cores + ((size_t)st.x * 2 + (bit ^ 1)) * (CHI * CHI) + tile, lane);
      }
    }
  };
  auto compute = [&](const Frags& F, int item) {
    const int s = item / NIS, ig = item % NIS;
    const int4 st = sched[s];
    const int k = st.x, nact = st.z, odd = st.w;
    // the other slice only serves the odd row, which most steps of a row
    // group do not have: its codes are decoded only when it does
    const int oin = odd >= 0 ? (odd & 0xffff) : -1, oout = odd >> 16;
    Frag<ER, KPL> Fm[MTI], Fo[MTI];
    if constexpr (kDec) {
#pragma unroll
      for (int q = 0; q < MTI; ++q) D::template decode<KPL>(F.m[q], Fm[q]);
      if (oin >= 0) {
#pragma unroll
        for (int q = 0; q < MTI; ++q) D::template decode<KPL>(F.o[q], Fo[q]);
      }
    }
    auto fm = [&](int q) -> const Frag<ER, KPL>& {
      if constexpr (kDec) return Fm[q];
      else return F.m[q];
    };
    auto fo = [&](int q) -> const Frag<ER, KPL>& {
      if constexpr (kDec) return Fo[q];
      else return F.o[q];
    };
    const int cexp = cexp_p ? cexp_p[k] : 0;
    const int ntile = (nact + 15) >> 4;
    // rows are renormalised every kRenormEvery steps: between two, a row
    // grows by at most a factor chi per step (core entries below 1)
    const bool rn = (s % kRenormEvery) == 0;
    // With BF16 cores the odd row rides on the matrix cores too: when the
    // row tile holding its input comes by, the other slice is applied to the
    // same B operand and the column of that row kept (stored after the loop,
    // since the main loop may also write its output slot).  FP32 matrix ops
    // are 8x slower, so there it stays a vector-ALU dot product.
    f4 oacc[MTI];
    int oe = 0;
    for (int r = 0; r < ntile; ++r) {
      const int row = 16 * r + m;
      typename D::template BOp<KPL> bo;
      A::template load_b<KPL>(cur + row * RS, g, bo);
      const int e = rn ? A::template row_exp<KPL>(bo) : 0;
      const float sc = __builtin_amdgcn_ldexpf(1.f, -e);  // exact power of two
      if (ig == 0 && wv == 0 && g == 0) exn[row] = exc[row] + e + cexp;
#pragma unroll
      for (int q = 0; q < MTI; ++q) {
        f4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = DR::template mma<KPL>(fm(q), bo, acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] *= sc;
        A::store4(nxt + row * RS, g * KPL + 4 * (wv * MT + ig * MTI + q), acc);
      }
      if (ODD_MFMA && r == (oin >> 4)) {
        oe = e;
#pragma unroll
        for (int q = 0; q < MTI; ++q) {
          f4 acc = {0.f, 0.f, 0.f, 0.f};
          acc = DR::template mma<KPL>(fo(q), bo, acc);
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[i] *= sc;
          oacc[q] = acc;
        }
      }
    }
    if (ODD_MFMA && oin >= 0) {  // lanes of column oin % 16 hold 4 output features each
      if (m == (oin & 15)) {
#pragma unroll
        for (int q = 0; q < MTI; ++q) A::store4(nxt + oout * RS, g * KPL + 4 * (wv * MT + ig * MTI + q), oacc[q]);
      }
      if (ig == 0 && wv == 0 && lane == (oin & 15)) exn[oout] = exc[oin] + oe + cexp;
    }
    if (!ODD_MFMA && oin >= 0) {  // FP32: the odd row as a vector-ALU dot product per output
      float v[KPL];
      A::template load_f32<KPL>(cur + oin * RS, g, v);
      int e = 0;
      if (rn) {
        float mx = 0.f;
#pragma unroll
        for (int c = 0; c < KPL; ++c) mx = fmaxf(mx, fabsf(v[c]));
        mx = group_max(mx);
        e = (mx > 0.f) ? __builtin_amdgcn_frexp_expf(mx) : 0;
      }
#pragma unroll
      for (int q = 0; q < MTI; ++q) {
        float p = 0.f;
#pragma unroll
        for (int c = 0; c < KPL; ++c) p = fmaf(__uint_as_float(F.o[q].w[c]), v[c], p);
        p += __shfl_xor(p, 16);
        p += __shfl_xor(p, 32);
        if (g == 0) A::store1(nxt + oout * RS, (m >> 2) * KPL + 4 * (wv * MT + ig * MTI + q) + (m & 3), __builtin_amdgcn_ldexpf(p, -e));
      }
      if (ig == 0 && wv == 0 && lane == 0) exn[oout] = exc[oin] + e + cexp;
    }
    if (ig == NIS - 1) {
      lds_barrier();
      float* tp = cur; cur = nxt; nxt = tp;
      int* te = exc; exc = exn; exn = te;
    }
  };
  // A ring of PFP fragment sets: loads run PFP - 1 items ahead of the
  // matrix ops, issued on every path (clamped to the last item) so that the
  // wait before the matrix ops never covers an item still being prefetched.
  // Two sets everywhere: a third (the FP8 sets are half the registers of
  // BF16 ones) measured slower at bond 256, and at bond 128 it costs the
  // kernel its second wave per SIMD.
  constexpr int PFP = (kDec && CHI == 256) ? PASS_PF_FP8 : 2;
  Frags FR[PFP];
  if (n_items > 0) {
#pragma unroll
    for (int q = 0; q < PFP - 1; ++q) load(FR[q], min(q, n_items - 1));
    for (int i = 0; i < n_items; i += PFP) {
#pragma unroll
      for (int r = 0; r < PFP; ++r) {
        if (i + r >= n_items) break;
        load(FR[(r + PFP - 1) % PFP], min(i + r + PFP - 1, n_items - 1));
        compute(FR[r], i + r);
      }
    }
  }
  __syncthreads();

  if (w_raw < a.W) {
    float* ov = a.out_vec + (((size_t)ty * a.W + w) * nslot) * CHI;
    for (int i = tid_w; i < nslot * CHI; i += NT_W) ov[i] = A::get(cur + (i / CHI) * RS, i % CHI);
    int32_t* oe = a.out_exp + ((size_t)ty * a.W + w) * nslot;
    for (int i = tid_w; i < nslot; i += NT_W) oe[i] = exc[i];
  }
}

template <class D, int CHI>
__global__ void __launch_bounds__(256, (pass_min_blocks<D, CHI>())) pass_kernel(PassArgs a) {
  pass_body<D, CHI>(a, blockIdx.x, blockIdx.y);  // y = term * ng + group
}

// ============================================================================
// sampler arguments (rtt_chain.hpp)
// ============================================================================
struct ChainArgs {
  const void* cores;         // [T][L][2][CHI*CHI] forward fragment layout (prescaled)
  const void* cores_bwd;     // [T][L][2][CHI*CHI] backward fragment layout (prescaled)
  const int32_t* cesum;      // [T][L+1] prefix sums of the per-position scale exponents
  const int32_t* pi;         // [L]
  const uint64_t* rmask;     // [N][LW] bit k set iff position k reads spin j
  const int32_t* order;      // [N] proposal order
  const int32_t* first;      // [N] first position of spin j, -1 if none
  const int32_t* last;       // [N] last position of spin j, -1 if none
  const double* coeffs;      // [T]
  int T, L, N, nw, LW, W;
  uint64_t* spins;
  double* logabs; int8_t* sign; uint32_t* accepts; int32_t* status;
  uint64_t seed, rstream, sweep0;
  int n_sweeps;
  int mode;                  // 0: amplitudes only, 1: sweeps
  // Column checkpoints (sweeps): the right environments of bonds
  // ck_first + i * ck_step, i < n_ck, for the current configuration, with a
  // per-walker validity mask (0: none); kept in LDS, or in global memory
  // (ckg: [block][2 buffers][n_ck][T] vectors) with bond 256.
  int n_ck, ck_first, ck_step;
  void* ckg;
  int ck_cap;                // checkpoints there is room for in ckg
  void* pg;                  // prefixes in global memory ([block][T][2] vectors), or null
};

// ============================================================================
// persistent forms for batches of RTTs
// ============================================================================
// Work items (int4): x = descriptor index, y = block index within that
// descriptor's launch, z = term (pass kernel).  Blocks take items from a
// device counter until the list is exhausted; every wave reaches the exit.
__device__ __forceinline__ int next_item(int* counter, int* s_item) {
  if (threadIdx.x == 0) *s_item = atomicAdd(counter, 1);
  __syncthreads();
  const int it = *s_item;
  __syncthreads();
  return it;
}

// (Up to bond 64 with both forms compiled in: 256 registers and, at 64, 100
// bytes of scratch in BF16 and 48 in FP8, where the rows-in-LDS form alone took
// 119.  Members that still take that form lose nothing by it: eight of 10x10,
// 600 to 691 walkers, bond 64 BF16, 6.09 ms of passes against 6.23.)
template <class D, int CHI>
__global__ void __launch_bounds__(256, (pass_wave_bond<D, CHI>() ? 2 : pass_min_blocks<D, CHI>()))
    pass_persistent(const PassArgs* descs, const int4* items, int n_items, int* counter) {
  __shared__ int s_item;
  for (;;) {
    const int it = next_item(counter, &s_item);
    if (it >= n_items) break;
    const int4 w = items[it];
    const PassArgs a = descs[w.x];
    if constexpr (pass_wave_bond<D, CHI>()) {
      if (a.wave) pass_wave_any<D, CHI>(a, w.y, w.z);
      else pass_body<D, CHI>(a, w.y, w.z);
    } else {
      pass_body<D, CHI>(a, w.y, w.z);
    }
    __syncthreads();
  }
}

}  // namespace rttk
