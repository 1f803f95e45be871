// Sampler kernels: amplitudes and Metropolis sweeps, 16 walkers per matrix-core column group.
//
// Every amplitude is contracted from both ends at once: one set of waves
// carries row vectors from the left (forward fragments), another column
// vectors from the right (backward fragments, from the boundary or from a
// checkpoint); they meet half way and are joined by an FP64 dot product.
//
// A vector is kept the way the matrix ops hand it over: lane (g, m) of a wave
// produces features g chi/4 + 4 t .. + 3 of walker m from output tile t (the
// fragments' row order is chosen for that) and consumes exactly the features
// [g chi/4, (g + 1) chi/4) of walker m in the next step.  So
//   * up to bond 64 one wave carries all features of its 16 walkers and the
//     vectors never leave its registers: no LDS traffic and no barrier
//     between the steps of a contraction;
//   * wider bonds split the features over SW waves, which exchange their
//     tiles lane to lane through LDS (16-byte accesses, conflict-free).
#pragma once
#include <float.h>
#include <limits.h>
#include <math.h>

#include "rtt_kernels.hpp"
#include "rtt_tile.hpp"

namespace rttk {

// Waves per side SW.  One where a step (both slices, all features) is short
// enough for it: BF16 and FP8 up to bond 64 (32 matrix ops), FP32 at 16.  FP32
// matrix ops run at an eighth of the rate, so bond 64 uses four waves (sweep of
// 4096 walkers at 8x8: 3.00 ms, with two 3.77) and 128 two (four would halve
// the registers: 9.1 against 5.0 ms at 6x6, 1000 walkers).  Bond 32 uses two
// (6x6, 1000 walkers: 0.45 ms, with one 0.54; in a batch, six states of 300 to
// 365, 0.98 against 1.15), and one where two terms advance side by side (two
// terms: 0.57 against 0.82).  BF16 and FP8 use two from 128 on, for 16 and 32
// walkers alike: the waves' partial dot products then meet in one order
// whatever the block's size.
template <class D, int CHI, int CG = 1, int TW = 1>
struct SampGeo {
  static constexpr int SW = D::kF32 ? (CHI == 128 ? 2 : CHI == 64 ? 4 : CHI == 32 && TW == 1 ? 2 : 1) : (CHI >= 128 ? 2 : 1);
  // parts of a wave's dot product, added as the waves' are: as many in all at
  // one bond, so that every shape of block gives the same bits
  static constexpr int DP = D::kF32 && CHI == 32 ? 2 / SW : 1;
  static constexpr int NV = CHI / 16;  // tiles of a vector = 16-byte words per lane
  static constexpr int MT = NV / SW;   // output tiles per wave
  // fragment slots (tiles) in flight per wave: two steps up to bond 64 and
  // for 16 walkers at 128, else about what the registers beside the vectors
  // hold (a step of bond 256 is 256 or 512 matrix ops; eight slots there, or
  // four of FP32 at 128, took 2.4 times as long).  Blocks of 32 at bond 256
  // spill even with two, 736 bytes a lane, and are still the faster: 9x9, two
  // terms, 50.7 ms a sweep of 8000 walkers against 56.2 in blocks of 16.
  static constexpr int NS = CHI <= 64 || (CHI == 128 && CG == 1 && !D::kF32) ? 2 * MT
                            : CHI == 128 ? (D::kF32 ? 2 : MT) : sizeof(typename D::elem) == 1 ? 4 / CG : 2;
};

// waves per SIMD the sampler is compiled for (a register budget): two up to
// bond 64, where 256 registers hold everything and results of matrix ops
// then stay in ordinary vector registers
template <class D, int CHI>
constexpr int samp_min_waves() { return CHI <= 64 ? 2 : 1; }

// words (16 bytes per lane) of one 16-walker vector
template <int CHI>
constexpr int kRowWords = CHI / 16 * 64;

// LDS layout of one block (byte offsets).  Vectors are [tile][lane] 16-byte
// words.  P: the prefix of each term; PU: with split, the other slice's
// product of a proposal's first step; XB: the step buffers (rows and columns,
// two each) when a side has several waves, else the columns handed to the
// row wave; CK: column checkpoints, saved and candidate.
struct SampLayout {
  int pb, xb, ck, vec_end, ep, ec, cke, fexp, fval, ub, pm, sp, total;
  bool split;
  __host__ __device__ SampLayout(int chi, int T, int LW, int nw, int cg, int sw, int tw, int nck, bool ck_lds,
                                 bool p_lds) {
    const int nb = 16 * cg, row = chi * 64 * cg;
    const int nx = sw > 1 ? 4 : tw;
    const int cks = 2 * nck * T;  // checkpoint vectors, saved and candidate
    const int tail = (2 * T + tw + cks) * nb * 4 + T * sw * nb * 8 + kUAhead * nb * 8 + nb * (LW + nw) * 8 + 64;
    split = !p_lds || (2 * T + nx + (ck_lds ? cks : 0)) * row + tail <= kLds;
    pb = 0;
    xb = p_lds ? (split ? 2 : 1) * T * row : 0;
    ck = xb + nx * row;
    vec_end = ck + (ck_lds ? cks * row : 0);
    fval = vec_end;                     // double [T][sw][nb] partial dot products
    ub = fval + T * sw * nb * 8;        // double [kUAhead][nb] uniforms of the next proposals
    pm = ub + kUAhead * nb * 8;         // uint64 [nb][LW] position bits
    sp = pm + nb * LW * 8;              // uint64 [nb][nw] spins
    ep = sp + nb * nw * 8;              // int [T][nb] prefix exponents
    ec = ep + T * nb * 4;               // int [tw][nb] column exponents
    fexp = ec + tw * nb * 4;            // int [T][nb] amplitude exponents
    cke = fexp + T * nb * 4;            // int [2][nck][T][nb] checkpoint exponents
    total = cke + cks * nb * 4;
  }
  static constexpr int kLds = 160 * 1024;
  static constexpr int kUAhead = 16;
};

// ---------------------------------------------------------------- sampler body
// Block of 2 * SW * TW waves for 16 * CG walkers: TW terms of a combination
// advance at the same time (the others take turns).  CKP compiles column
// checkpoints in, CKG keeps their vectors in global memory, PG the prefixes.
template <class D, int CHI, int CG, int TW, bool CKP, bool CKG, bool PG>
__device__ __forceinline__ void samp_body(const ChainArgs& a, int bx, uint64_t sweep0) {
  using E = typename D::elem;
  using G = SampGeo<D, CHI, CG, TW>;
  using Op = TileOp<D, CHI>;
  constexpr int SW = G::SW, NV = G::NV, MT = G::MT, NS = G::NS, KPL = CHI / 4;
  constexpr int NB = 16 * CG, ROW = kRowWords<CHI>;
  constexpr bool VAR = CKP && CG > 1;  // column groups may start and meet at bonds of their own
  constexpr bool ONE = SW > 1 && !(CHI == 256 && CG == 2);  // a step is one piece of code
  constexpr int DU = NS > MT ? NS / MT : 1;             // steps of fragments in flight
  constexpr int UN = DU % 2 ? DU : DU / 2;              // pairs of steps unrolled
  static_assert(NS % MT == 0 || MT % NS == 0, "the ring divides a step, or steps the ring");
  static_assert(D::kF32 || MT % 2 == 0, "hi and lo words pair two tiles");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lane = threadIdx.x & 63;
  // wave-uniform, so that every address below is a scalar plus 16 lane
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave % SW, side = (wave / SW) & 1, tw = wave / (2 * SW);
  const int g = lane >> 4, m = lane & 15;
  const int nthr = blockDim.x;
  const int T = a.T, L = a.L, LW = a.LW, nw = a.nw;
  const int NCK = CKP ? a.n_ck : 0;
  const SampLayout lay(CHI, T, LW, nw, CG, SW, TW, NCK, !CKG, !PG);
  const bool split = lay.split;
  u32x4* pbuf_l = reinterpret_cast<u32x4*>(lds_raw + lay.pb) + lane;
  u32x4* pbuf_g = PG ? reinterpret_cast<u32x4*>(a.pg) + (size_t)bx * 2 * T * CG * ROW + lane : nullptr;
  u32x4* xbuf = reinterpret_cast<u32x4*>(lds_raw + lay.xb) + lane;
  u32x4* ckbuf_l = reinterpret_cast<u32x4*>(lds_raw + lay.ck) + lane;
  u32x4* ckbuf_g = CKG ? reinterpret_cast<u32x4*>(a.ckg) + (size_t)bx * 2 * NCK * T * CG * ROW + lane : nullptr;
  double* fval = reinterpret_cast<double*>(lds_raw + lay.fval);
  double* ub = reinterpret_cast<double*>(lds_raw + lay.ub);
  uint64_t* pm = reinterpret_cast<uint64_t*>(lds_raw + lay.pm);
  uint64_t* sp = reinterpret_cast<uint64_t*>(lds_raw + lay.sp);
  int* ep = reinterpret_cast<int*>(lds_raw + lay.ep);
  int* ec = reinterpret_cast<int*>(lds_raw + lay.ec);
  int* fexp = reinterpret_cast<int*>(lds_raw + lay.fexp);
  int* cke = reinterpret_cast<int*>(lds_raw + lay.cke);

  // prefix buffer `which` of term t (word 0 of this lane); with split, buffer
  // 0 holds the flipped and 1 the unflipped extension, chosen per walker by
  // psel (accepted or not) when the next proposal reads it
  auto pword = [&](int t, int which, int cg) {
    const int o = ((t * (split ? 2 : 1) + which) * CG + cg) * ROW;
    if constexpr (PG) return pbuf_g + o;
    else return pbuf_l + o;
  };
  auto xword = [&](int b, int cg) { return xbuf + (b * CG + cg) * ROW; };
  auto ckword = [&](int which, int i, int t, int cg) { return ((which * NCK + i) * T + t) * CG * ROW + cg * ROW; };
  auto ckexp = [&](int which, int i, int t, int wn) -> int& { return cke[((which * NCK + i) * T + t) * NB + wn]; };
  // index of the first checkpoint whose bond is >= b (NCK if none)
  auto ck_ceil = [&](int b) {
    const int d = b - a.ck_first;
    return d <= 0 ? 0 : min(NCK, (d + a.ck_step - 1) / a.ck_step);
  };
  auto ck_bits = [](int lo, int hi) -> uint32_t {  // bits [lo, hi)
    return hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
  };
  auto ck_bond = [&](int i) { return a.ck_first + i * a.ck_step; };
  auto rword = [&](int j, int wd) -> uint64_t { return uniform_load(a.rmask, (long long)j * LW + wd); };

  const int w0 = bx * NB;
  bool live[CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) live[cg] = (w0 + 16 * cg + m) < a.W;
  for (int i = threadIdx.x; i < NB * nw; i += nthr) {
    const int n = i / nw, wd = i % nw;
    sp[i] = (w0 + n < a.W) ? a.spins[(size_t)(w0 + n) * nw + wd] : 0ull;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NB * LW; i += nthr) {
    const int n = i / LW, wd = i % LW;
    uint64_t word = 0;
    for (int b = 0; b < 64 && 64 * wd + b < L; ++b) {
      const int q = a.pi[64 * wd + b];
      word |= (uint64_t)spin_bit(sp + n * nw, q) << b;
    }
    pm[i] = word;
  }
  __syncthreads();

  const char* cores = static_cast<const char*>(side == 0 ? a.cores : a.cores_bwd);
  constexpr size_t SLICE = (size_t)CHI * CHI * sizeof(E);
  constexpr int TILE = 64 * KPL * (int)sizeof(E);
  uint32_t csel[CG];   // per checkpoint: which of its two buffers is the saved one
  int psel[CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) { csel[cg] = 0; psel[cg] = 0; }

  u32x4 r[CG][NV];     // the vector a step consumes
  u32x4 o[CG][MT];     // this wave's tiles of the vector it produced
  u32x4 oth[CG][MT];   // with split: the other slice's product of the first step
  int ex[CG], exf[CG]; // exponent of the running vector, and after the first step

  // Term t: rows (side 0) from the prefix at bond k0 to bond kc[cg], columns
  // from bond ks[cg] (the right boundary if L, else the saved column of that
  // checkpoint) down to kc[cg], with spin jflip flipped (-1: none).  Columns
  // reaching a checkpoint bond are kept: as its saved column when the bond
  // lies past lj, the last position of the flipped spin (they are then the
  // current configuration's), else as its candidate.  Vectors are scaled by a
  // power of two every kRenormEvery steps (exact), exponents summed in ex.
  // One wave per side: the result is r.  Several: the result is in step
  // buffer 2 side + (parity of the last step), every step ends with a block
  // barrier and the side with fewer steps takes part in the other's.
  auto segment = [&](int t, int k0, const int (&kc)[CG], const int (&ks)[CG], bool cols, int lj, int jflip,
                     bool sp0) {
    int n = 0, nmax = 0, kbeg = k0, s0[CG], s1[CG];  // steps of this side; group cg runs [s0, s1)
    {
      int top = ks[0];
      if constexpr (VAR) top = max(ks[0], ks[CG - 1]);
      if (side == 1) kbeg = top - 1;
      int nr = 0, nc = 0;
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) {
        const int q = VAR ? cg : 0;
        nr = max(nr, kc[q] - k0);
        nc = cols ? max(nc, top - kc[q]) : 0;
        s0[cg] = side == 0 ? 0 : top - ks[q];
        s1[cg] = side == 0 ? kc[q] - k0 : (cols ? top - kc[q] : 0);
      }
      n = __builtin_amdgcn_readfirstlane(side == 0 ? nr : nc);
      nmax = __builtin_amdgcn_readfirstlane(max(nr, nc));
      kbeg = __builtin_amdgcn_readfirstlane(kbeg);
    }
    const int dk = side == 0 ? 1 : -1;
    const char* base = uniform_ptr(cores + ((size_t)t * L + kbeg) * 2 * SLICE + (size_t)wv * MT * TILE);
    const long long kstep = dk * 2 * (long long)SLICE;
    Frag<E, KPL> S[NS][2];
    auto load = [&](Frag<E, KPL>(&f)[2], int i, int mt) {
      // (the bases stay scalar: an offset the instruction cannot hold would
      // otherwise become a 64-bit vector addition per load)
      typedef const __attribute__((address_space(1))) char* gchar;
      constexpr int WIN = 4096;  // reach of the instruction's offset
      gchar p = (gchar)(uintptr_t)(base + (long long)min(i, n - 1) * kstep + mt * TILE / WIN * WIN);
      gchar q = p + SLICE;
      asm("" : "+s"(p));
      asm("" : "+s"(q));
      load_frag2<E, KPL, CG == 1>(f, p + mt * TILE % WIN, q + mt * TILE % WIN, lane);
    };
    if (n > 0) {
#pragma unroll
      for (int q = 0; q < (SW == 1 ? NS - MT : NS); ++q) load(S[q], q / MT, q % MT);
    }
    // the starting vector of group cg into the words dst[v]
    auto source = [&](int cg, u32x4(&dst)[NV]) {
      const int q = VAR ? cg : 0;
      if (side == 0 ? k0 == 0 : ks[q] == L) {
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[v] = u32x4{0, 0, 0, 0};
        dst[0][0] = g == 0 ? Op::kUnit : 0u;
        ex[cg] = 0;
      } else if (side == 0) {
        const u32x4* s = pword(t, 0, cg) + (split && psel[cg] ? CG * ROW : 0);
#pragma unroll
        for (int v = 0; v < NV; ++v) dst[v] = s[v * 64];
        ex[cg] = ep[t * NB + 16 * cg + m];
      } else if constexpr (CKP) {
        const int i = (ks[q] - a.ck_first) / a.ck_step, which = (csel[cg] >> i) & 1;
        const int w = ckword(0, i, t, cg) + (which ? NCK * T * CG * ROW : 0);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if constexpr (CKG) dst[v] = __builtin_nontemporal_load(ckbuf_g + w + v * 64);
          else dst[v] = ckbuf_l[w + v * 64];
        }
        ex[cg] = ckexp(which, i, t, 16 * cg + m);
      }
    };
    if constexpr (SW == 1) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) source(cg, r[cg]);
    }
    // the next checkpoint the columns reach (bond ckb, index cki; -1: none)
    int cki = -1, ckb = -1;
    if (CKP && side == 1 && NCK > 0 && kbeg >= a.ck_first) {
      cki = min(NCK - 1, (kbeg - a.ck_first) / a.ck_step);
      ckb = a.ck_first + cki * a.ck_step;
    }
    // slice bits of the next kRenormEvery positions, the first in bit 0
    uint32_t win[CG];
    auto window = [&](int i) {
      const int k = kbeg + dk * i, lo = side == 0 ? k : max(0, k - (kRenormEvery - 1));
      const int wd = lo >> 6, wd1 = min(wd + 1, LW - 1);
      const uint64_t f0 = jflip >= 0 ? rword(jflip, wd) : 0ull, f1 = jflip >= 0 ? rword(jflip, wd1) : 0ull;
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) {
        const uint64_t* p = pm + (16 * cg + m) * LW;
        const uint64_t w0b = p[wd] ^ f0, w1b = p[wd1] ^ f1;
        const int sh = lo & 63;
        const uint32_t up = (uint32_t)((w0b >> sh) | (sh ? w1b << (64 - sh) : 0ull));  // bit q: position lo + q
        win[cg] = side == 0 ? up : __brev(up) >> (31 - (k - lo));
      }
    };
    // One step: out = this wave's tiles of (in times the walkers' slices).
    // With several waves per side the ring is refilled inside the step, which
    // then is one piece of code (ONE): with a copy for steps that renormalise
    // (rn) and one for those that also keep the other slice's product (spl),
    // the fragments in flight were moved to common registers where the copies
    // met, and all of them waited for (BF16 bond 128, 10x10, 8192 walkers: 26.9
    // -> 24.3 ms a sweep; FP8 bond 256, 8x8, 300 walkers: 11.9 -> 10.0 ms).
    // Blocks of 32 at bond 256 keep the copies: their sums leave no room for
    // the tests between tiles (9x9, two terms, 8192 walkers: 49.8 ms against 55.1).
    auto step = [&](auto rnc, auto spc, auto dc, int i, bool rn, bool spl, const u32x4(&in)[CG][NV],
                    u32x4(&out)[CG][MT]) {
      constexpr bool RN = decltype(rnc)::value, SPL = decltype(spc)::value;
      constexpr int DD = decltype(dc)::value;
      if constexpr (RN) {
        if (i % kRenormEvery == 0) window(i);
      }
      bool bit[CG];
      float psc[CG];
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) {
        bit[cg] = (win[cg] >> (i % kRenormEvery)) & 1u;
        if constexpr (ONE) psc[cg] = 1.f;
        if constexpr (RN) {
          if (!ONE || rn) {
            const int e = Op::row_exp(in[cg]);
            psc[cg] = __builtin_amdgcn_ldexpf(1.f, -e);  // exact power of two
            if (!VAR || (i >= s0[cg] && i < s1[cg])) ex[cg] += e;
          }
        }
      }
      // tile mt's products: acc[mt % NA]; the tile before is selected and split
      // between its matrix ops, and each chunk decoded during the one before
      // The written order is held only with FP8 codes at bond 256, where the
      // decode fills the matrix ops' shadow (9x9, two terms, 8192 walkers:
      // 48.8 ms a sweep, 51.3 left to the scheduler); elsewhere holding it cost
      // more than it hid (8x8 BF16 1.40 against 1.34 ms, FP32 3.77 against 3.04).
      constexpr bool HOLD = sizeof(E) == 1 && CHI == 256;
      constexpr int OPT = Op::NCH * Op::OPC * 2 * CG;  // matrix ops per tile
      constexpr int NST = Op::kStages * CG;            // pieces of vector work per tile
      constexpr int OPCH = Op::OPC * 2 * CG, NPC = 2 * Op::kPieces;
      // (sums of all tiles are kept where one test after them serves spl)
      constexpr int NA = ONE && CG == 1 ? MT : 2;
      f4 acc[NA][2][CG];
      typename Op::Operand x[2][2];
      typename Op::Post pst, psu;
      auto finish = [&](int mt, int st) {  // piece st of tile mt's vector work
        const int cg = st / Op::kStages, q = st % Op::kStages, b = mt % NA;
        Op::template post<RN, MT>(q, pst, bit[cg], acc[b][0][cg], acc[b][1][cg], RN ? psc[cg] : 1.f, out[cg], mt);
        if constexpr (SPL)
          Op::template post<RN, MT>(q, psu, !bit[cg], acc[b][0][cg], acc[b][1][cg], psc[cg], oth[cg], mt);
      };
      // the other slice's product of tiles [lo, hi)
      auto finish_other = [&](int lo, int hi) {
        if constexpr (ONE) {
          int f = __builtin_amdgcn_readfirstlane((int)spl);
          asm("" : "+s"(f));  // (a test here, not a copy of the rest of the step)
          if (f)
#pragma unroll
            for (int mt = lo; mt < hi; ++mt)
#pragma unroll
              for (int st = 0; st < NST; ++st) {
                const int cg = st / Op::kStages, b = mt % NA;
                Op::template post<RN, MT>(st % Op::kStages, psu, !bit[cg], acc[b][0][cg], acc[b][1][cg], psc[cg], oth[cg], mt);
              }
        }
      };
      auto frag = [&](int mt) -> Frag<E, KPL>(&)[2] { return S[(DD * MT + mt) % NS]; };
#pragma unroll
      for (int q = 0; q < NPC; ++q) Op::decode(frag(0)[q / Op::kPieces], 0, q % Op::kPieces, x[0][q / Op::kPieces]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int c = 0; c < Op::NCH; ++c) {
          const int xb = (mt * Op::NCH + c) % 2;
          const bool lastc = c == Op::NCH - 1;
#pragma unroll
          for (int u = 0; u < OPCH; ++u) {
            const int kk = u / (2 * CG), sl = u / CG % 2, cg = u % CG;
            f4& A = acc[mt % NA][sl][cg];
            if (c == 0 && kk == 0) A = f4{0.f, 0.f, 0.f, 0.f};
            A = Op::op(x[xb][sl], in[cg], c, kk, A);
            // decode of the next chunk (of the next tile after the last one)
            if (!(lastc && mt == MT - 1)) {
#pragma unroll
              for (int q = u * NPC / OPCH; q < (u + 1) * NPC / OPCH; ++q)
                Op::decode(frag(lastc ? mt + 1 : mt)[q / Op::kPieces], lastc ? 0 : c + 1, q % Op::kPieces,
                           x[xb ^ 1][q / Op::kPieces]);
            }
            if (mt > 0) {
              const int w = c * OPCH + u;
#pragma unroll
              for (int st = w * NST / OPT; st < (w + 1) * NST / OPT; ++st) finish(mt - 1, st);
            }
            if constexpr (HOLD) hold_order();
          }
        }
        if constexpr (SW > 1) {  // the slot is free: the tile NS places further on
          load(frag(mt), i + (mt + NS) / MT, (mt + NS) % MT);
          hold_loads();
        }
        if (NA == 2 && mt > 0) finish_other(mt - 1, mt);
      }
#pragma unroll
      for (int st = 0; st < NST; ++st) finish(MT - 1, st);
      finish_other(NA == 2 ? MT - 1 : 0, MT);
    };
    // fragments of the step DU - 1 ahead, into the slots of the last step (one
    // wave per side)
    auto ahead = [&](auto dc, int i) {
      if constexpr (SW == 1) {
        constexpr int DN = (decltype(dc)::value + DU - 1) % DU;
#pragma unroll
        for (int q = 0; q < MT; ++q) load(S[DN * MT + q], i + DU - 1, q);
        hold_order();
      }
    };
    auto run = [&](auto dc, int i, const u32x4(&in)[CG][NV], u32x4(&out)[CG][MT]) {
      ahead(dc, i);
      bool rn = i % kRenormEvery == 0;
      if constexpr (VAR)
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) rn |= i == s0[cg];
      auto spl = [&]() { return i == 0 && sp0 && side == 0; };
      if constexpr (ONE) {
        step(std::true_type{}, std::false_type{}, dc, i, rn, spl(), in, out);
      } else {
        // (asked for beforehand with BF16 and FP8 cores and one wave per side,
        // 5x5 sweeps 1-2% shorter; with FP32, and in blocks of 32 at bond 256,
        // 1% longer)
        constexpr bool EARLY = SW == 1 && !D::kF32;
        bool first = false;
        if constexpr (EARLY) first = spl();
        if (!rn) step(std::false_type{}, std::false_type{}, dc, i, false, false, in, out);
        else if (EARLY ? first : spl()) step(std::true_type{}, std::true_type{}, dc, i, true, true, in, out);
        else step(std::true_type{}, std::false_type{}, dc, i, true, false, in, out);
      }
    };
    // after step i: the two extensions of the prefix, and checkpoints passed
    auto keep = [&](int i, const u32x4(&out)[CG][MT]) {
      if (i == 0 && sp0 && side == 0) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          u32x4* d = pword(t, 0, cg) + wv * MT * 64;
#pragma unroll
          for (int v = 0; v < MT; ++v) {
            d[v * 64] = out[cg][v];
            d[v * 64 + CG * ROW] = oth[cg][v];
          }
          exf[cg] = ex[cg];
        }
      }
      if constexpr (CKP) {
        const int k = kbeg + dk * i;
        if (side == 1 && k == ckb) {
#pragma unroll
          for (int cg = 0; cg < CG; ++cg) {
            if (VAR && !(i >= s0[cg] && i < s1[cg])) continue;
            const int which = ((csel[cg] >> cki) & 1) ^ (k > lj ? 0 : 1);
            const int w = ckword(0, cki, t, cg) + (which ? NCK * T * CG * ROW : 0) + wv * MT * 64;
#pragma unroll
            for (int v = 0; v < MT; ++v) {
              if constexpr (CKG) __builtin_nontemporal_store(out[cg][v], ckbuf_g + w + v * 64);
              else ckbuf_l[w + v * 64] = out[cg][v];
            }
            if (wv == 0 && g == 0) ckexp(which, cki, t, 16 * cg + m) = ex[cg];
          }
          --cki;
          ckb = cki >= 0 ? ckb - a.ck_step : -1;
        }
      }
    };
    if constexpr (SW == 1) {
      for (int i = 0; i < n; i += 2 * UN) {
        // (an odd ring depth needs twice as many steps unrolled for the
        // vectors to change places)
        bool more = true;
        auto two = [&](auto uc) {
          constexpr int U = decltype(uc)::value;
          if (!more) return;
          run(std::integral_constant<int, U % DU>{}, i + U, r, o);
          keep(i + U, o);
          if (i + U + 1 >= n) {
#pragma unroll
            for (int cg = 0; cg < CG; ++cg)
#pragma unroll
              for (int v = 0; v < NV; ++v) r[cg][v] = o[cg][v];
            more = false;
            return;
          }
          // (only even steps renormalise)
          constexpr std::integral_constant<int, (U + 1) % DU> dc{};
          ahead(dc, i + U + 1);
          step(std::false_type{}, std::false_type{}, dc, i + U + 1, false, false, o, r);
          keep(i + U + 1, r);
          if (i + U + 2 >= n) more = false;
        };
        two(std::integral_constant<int, 0>{});
        if constexpr (UN > 1) two(std::integral_constant<int, 2>{});
        if constexpr (UN > 2) two(std::integral_constant<int, 4>{});
        if (!more) break;
      }
    } else {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg)
        if (s0[cg] >= s1[cg]) {  // no step: the result is the starting vector
          source(cg, r[cg]);
          if (wv == 0)
#pragma unroll
            for (int v = 0; v < NV; ++v) xword(2 * side, cg)[v * 64] = r[cg][v];
        }
      auto one = [&](auto dc, int i) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          if (i == s0[VAR ? cg : 0]) source(cg, r[cg]);
          else {
            const u32x4* s = xword(2 * side + ((i - 1) & 1), cg);
#pragma unroll
            for (int v = 0; v < NV; ++v) r[cg][v] = s[v * 64];
          }
        }
        run(dc, i, r, o);
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          if (VAR && !(i >= s0[cg] && i < s1[cg])) continue;
          u32x4* d = xword(2 * side + (i & 1), cg) + wv * MT * 64;
#pragma unroll
          for (int v = 0; v < MT; ++v) d[v * 64] = o[cg][v];
        }
        lds_barrier();
        keep(i, o);
      };
      static_assert(DU <= 2, "one or two steps of fragments in flight");
      for (int i = 0; i < n; i += DU) {
        one(std::integral_constant<int, 0>{}, i);
        if constexpr (DU > 1) {
          if (i + 1 >= n) break;  // (not a path back to the loop with fewer loads in flight)
          one(std::integral_constant<int, 1>{}, i + 1);
        }
      }
      for (int i = n; i < nmax; ++i) lds_barrier();
    }
  };

  // barrier of everything the block exchanges (checkpoints and prefixes kept
  // in global memory included)
  auto block_sync = [&]() {
    if constexpr (CKG || PG) __syncthreads();
    else lds_barrier();
  };
  // Join rows and columns of the term each wave group has just contracted:
  // FP64 partial dot products per row wave, and the summed exponents.
  auto join = [&](int t, bool valid, int k0, const int (&kc)[CG], const int (&ks)[CG], bool sp0) {
    if (valid && side == 1) {
      if constexpr (SW == 1) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
#pragma unroll
          for (int v = 0; v < NV; ++v) xword(tw, cg)[v * 64] = r[cg][v];
      }
      if (wv == 0 && g == 0)
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) ec[tw * NB + 16 * cg + m] = ex[cg];
    }
    lds_barrier();
    if (valid && side == 0) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) {
        const int q = VAR ? cg : 0;
        u32x4 x[MT], y[MT];
        if constexpr (SW == 1) {
#pragma unroll
          for (int v = 0; v < MT; ++v) {
            x[v] = r[cg][v];
            y[v] = xword(tw, cg)[v * 64];
          }
        } else {
          int top = ks[0];
          if constexpr (VAR) top = max(ks[0], ks[CG - 1]);
          const int pr = kc[q] > k0 ? (kc[q] - k0 - 1) & 1 : 0, pc = ks[q] > kc[q] ? (top - kc[q] - 1) & 1 : 0;
#pragma unroll
          for (int v = 0; v < MT; ++v) {
            x[v] = xword(pr, cg)[(wv * MT + v) * 64];
            y[v] = xword(2 + pc, cg)[(wv * MT + v) * 64];
          }
        }
        double s = 0.0;
#pragma unroll
        for (int p = 0; p < G::DP; ++p) {
          constexpr int PW = MT / G::DP;
          u32x4 xp[PW], yp[PW];
#pragma unroll
          for (int v = 0; v < PW; ++v) {
            xp[v] = x[p * PW + v];
            yp[v] = y[p * PW + v];
          }
          double d = Op::template dot<PW>(xp, yp);
          d += __shfl_xor(d, 16);
          d += __shfl_xor(d, 32);
          s = p == 0 ? d : s + d;
        }
        if (g == 0) {
          const int wn = 16 * cg + m;
          fval[(t * SW + wv) * NB + wn] = s;
          if (wv == 0) {
            fexp[t * NB + wn] = ex[cg] + ec[tw * NB + wn] + uniform_load(a.cesum, (long long)t * (L + 1) + L);
            if (sp0) ep[t * NB + wn] = exf[cg];
          }
        }
      }
    }
    block_sync();
  };
  // combined amplitude of walker slot wn from the recorded values: mantissa in
  // [0.5, 1) and exponent; 0 if it vanishes, -1 if it is not finite (every
  // lane of every wave computes it for its walkers)
  auto amp = [&](int wn, double& mant, int& e2) -> int {
    // value of term t: m 2^e (read twice rather than kept in an indexed array,
    // which would live in scratch memory)
    auto term = [&](int t, double& v, int& e) {
      double f = fval[t * SW * NB + wn];
#pragma unroll
      for (int q = 1; q < SW; ++q) f += fval[(t * SW + q) * NB + wn];
      int ed = 0;
      const double md = frexp(f, &ed);
      v = uniform_load(a.coeffs, t) * md;
      e = fexp[t * NB + wn] + ed;
    };
    double v, S = 0.0;
    int e, emax = INT_MIN, eS = 0;
    for (int t = 0; t < T; ++t) {
      term(t, v, e);
      if (v != 0.0 && e > emax) emax = e;
    }
    mant = 0.0;
    e2 = 0;
    if (emax == INT_MIN) return 0;
    if (T == 1) {
      S = v;
    } else {
      for (int t = 0; t < T; ++t) {
        term(t, v, e);
        if (v != 0.0) S += ldexp(v, e - emax);
      }
    }
    mant = frexp(S, &eS);
    e2 = emax + eS;
    return mant == 0.0 ? 0 : isfinite(mant) ? 1 : -1;
  };
  // the meeting bond of a contraction over positions [f, ks)
  auto meet = [&](int f, int ks) { return f + (ks - f + 1) / 2; };

  // One loop over all contractions, so that the steps are compiled once: the
  // amplitude of the current configuration, then per proposal (if needed) the
  // prefix of every term brought up to the spin's first position, and the
  // flipped amplitude.  State of a walker is identical in all its lanes.
  enum { kInit, kAdvance, kPropose };
  double mcur[CG];
  int ecur[CG], stat[CG];
  uint32_t nacc[CG], vmask[CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) { mcur[cg] = 0.0; ecur[cg] = 0; stat[cg] = -5; nacc[cg] = 0; vmask[cg] = 0; }
  int task = kInit, ts = 0, qi = 0, pos = 0, filled = -1;
  bool behind = false;  // without split: the prefix still lacks the last decided spin
  while (true) {
    int j = -1, f = 0, lj = -1, il = 0, kk = 0;
    int kc[CG], ks[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) { ks[cg] = L; kc[cg] = meet(0, L); }
    if (task != kInit) {
      if (!behind && qi == a.N) {  // next sweep
        qi = 0;
        pos = 0;
        ++ts;
        filled = -1;
      }
      if (a.mode != 1 || ts >= a.n_sweeps) break;
      if (behind) {
        task = kAdvance;
        kk = pos + 1;
      } else {
        if (qi % SampLayout::kUAhead == 0 && filled != qi) {  // the uniforms of the next proposals
          filled = qi;
          lds_barrier();
          for (int i = threadIdx.x; i < SampLayout::kUAhead * NB; i += nthr) {
            const int q = qi + i / NB;
            if (q < a.N)
              ub[i] = philox_uniform(a.seed, a.rstream, (uint64_t)(w0 + i % NB), sweep0 + (uint64_t)ts,
                                     (uint64_t)a.order[q]);
          }
          lds_barrier();
        }
        j = uniform_load(a.order, qi);
        f = uniform_load(a.first, j);
        if (f < 0) {  // spin read by no position: ratio 1, always accepted
#pragma unroll
          for (int cg = 0; cg < CG; ++cg)
            if (live[cg] && stat[cg] == 0) {
              nacc[cg] += 1;
              if (wave == 0 && g == 0) sp[(16 * cg + m) * nw + (j >> 6)] ^= (1ull << (j & 63));
            }
          ++qi;
          continue;
        }
        task = pos < f ? kAdvance : kPropose;
        kk = f;
      }
      if (task == kAdvance) {
        j = -1;
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) kc[cg] = kk;
      } else {
        // the columns start from the first checkpoint past the spin's last
        // position that every walker of the group holds valid (else from the
        // right boundary)
        lj = uniform_load(a.last, j);
        il = ck_ceil(lj + 1);  // checkpoints below il lie at or before lj
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          if (CKP && NCK > 0) {
            uint32_t x = vmask[cg];
            x &= (uint32_t)__shfl_xor((int)x, 1);
            x &= (uint32_t)__shfl_xor((int)x, 2);
            x &= (uint32_t)__shfl_xor((int)x, 4);
            x &= (uint32_t)__shfl_xor((int)x, 8);
            const uint32_t elig = __builtin_amdgcn_readfirstlane(x & ~ck_bits(0, il));
            if (elig) ks[cg] = ck_bond(__builtin_ctz(elig));
          }
          kc[cg] = meet(f, ks[cg]);
        }
      }
    }
    // rows and columns meet half way; with split the first row step of a
    // proposal also leaves both extensions of the prefix through f
    const bool sp0 = split && task == kPropose;
    for (int tb = 0; tb < T; tb += TW) {
      const int t = tb + tw;
      const bool valid = TW == 1 || t < T;
      if (valid) segment(t, pos, kc, ks, task != kAdvance, lj, j, sp0);
      if (task != kAdvance) {
        join(t, valid, pos, kc, ks, sp0);
        continue;
      }
      if (valid && side == 0) {
#pragma unroll
        for (int cg = 0; cg < CG; ++cg) {
          u32x4* d = pword(t, 0, cg) + wv * MT * 64;
#pragma unroll
          for (int v = 0; v < MT; ++v) {
            if constexpr (SW == 1) d[v * 64] = r[cg][v];
            else d[v * 64] = o[cg][v];
          }
          if (wv == 0 && g == 0) ep[t * NB + 16 * cg + m] = ex[cg];
        }
      }
      block_sync();
    }
    if (task == kAdvance) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) psel[cg] = 0;
      pos = kk;
      behind = false;
      continue;
    }
    if (task == kInit) {
      // checkpoints the columns passed are valid (same mask in every lane of
      // a walker, in every wave)
      uint32_t v0 = 0;
      for (int i = 0; i < NCK; ++i)
        if (ck_bond(i) >= kc[0]) v0 |= 1u << i;
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) {
        vmask[cg] = v0;
        stat[cg] = amp(16 * cg + m, mcur[cg], ecur[cg]) == 1 ? 0 : -5;
      }
      task = kPropose;
      continue;
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      bool accept = false;
      if (live[cg] && stat[cg] == 0) {
        double mn;
        int en;
        const int ok = amp(16 * cg + m, mn, en);
        if (ok < 0) {
          stat[cg] = -5;
        } else if (ok == 1) {
          // u < (psi'/psi)^2 from mantissas and exponents
          const double u = ub[(qi % SampLayout::kUAhead) * NB + 16 * cg + m];
          const int de = max(-4000, min(4000, 2 * (en - ecur[cg])));
          if (u * (mcur[cg] * mcur[cg]) < ldexp(mn * mn, de)) {
            accept = true;
            mcur[cg] = mn;
            ecur[cg] = en;
            nacc[cg] += 1;
          }
        }
      }
      psel[cg] = split && !accept ? 1 : 0;
      // checkpoints: the columns computed past lj hold the current
      // configuration for every walker; those at or before lj become the
      // saved ones of the walkers that accepted (their two buffers change
      // places), and earlier ones at or before lj go stale for them
      if (CKP && NCK > 0) {
        const int ic0 = ck_ceil(kc[cg]), ic1 = ck_ceil(ks[cg]);  // computed: [ic0, ic1)
        const uint32_t cand = ck_bits(ic0, min(ic1, il)), stale = ck_bits(0, min(ic0, il));
        vmask[cg] |= ck_bits(max(ic0, il), ic1);
        if (accept) {
          vmask[cg] = (vmask[cg] | cand) & ~stale;
          csel[cg] ^= cand;
        }
      }
      if (wave == 0 && g == 0 && accept) {
        const int wn = 16 * cg + m;
        sp[wn * nw + (j >> 6)] ^= (1ull << (j & 63));
        for (int wd = 0; wd < LW; ++wd) pm[wn * LW + wd] ^= rword(j, wd);
      }
    }
    lds_barrier();
    ++qi;
    if (split) pos = f + 1;
    else behind = true;
  }

  // write back
  if (wave == 0 && g == 0) {
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      if (!live[cg]) continue;
      const int wn = 16 * cg + m;
      const int w = w0 + wn;
      if (a.mode == 1)
        for (int wd = 0; wd < nw; ++wd) a.spins[(size_t)w * nw + wd] = sp[wn * nw + wd];
      const bool ok = stat[cg] == 0;
      if (a.logabs) a.logabs[w] = ok ? log(fabs(mcur[cg])) + (double)ecur[cg] * 0.69314718055994530942 : NAN;
      if (a.sign) a.sign[w] = ok ? (mcur[cg] > 0 ? 1 : -1) : 0;
      if (a.accepts && a.mode == 1) a.accepts[w] += nacc[cg];
      if (a.status) a.status[w] = stat[cg];
    }
  }
}

template <class D, int CHI, int CG, int TW, bool CKP, bool CKG = false, bool PG = false>
__global__ void __launch_bounds__((2 * SampGeo<D, CHI, CG, TW>::SW * TW * 64), (samp_min_waves<D, CHI>()))
    chain_kernel(ChainArgs a) {
  samp_body<D, CHI, CG, TW, CKP, CKG, PG>(a, blockIdx.x, a.sweep0);
}

// Persistent form for batches; CG column groups of 16 walkers per item (the
// batch autotuner's tile choice).
template <class D, int CHI, int CG>
__global__ void __launch_bounds__((2 * SampGeo<D, CHI, CG>::SW * 64), (samp_min_waves<D, CHI>()))
    chain_persistent(const ChainArgs* descs, const int4* items, int n_items, int* counter, const uint64_t* sweep0) {
  __shared__ int s_item;
  for (;;) {
    // uniform item index: the descriptor's fields are then scalar loads
    const int it = __builtin_amdgcn_readfirstlane(next_item(counter, &s_item));
    if (it >= n_items) break;
    const int4 w = items[it];
    samp_body<D, CHI, CG, 1, false, false, false>(descs[w.x], w.y, *sweep0);
    __syncthreads();
  }
}

}  // namespace rttk
