// Tiles of vectors kept in registers: operations that the sampler
// (rtt_chain.hpp) and the wave-resident flip-ratio passes (rtt_kernels.hpp)
// share.  Lane (g, m) of a wave holds features [g chi/4, (g + 1) chi/4) of
// vector m, as the matrix ops leave them and take them.
#pragma once
#include "rtt_device.hpp"

namespace rttk {

// ---------------------------------------------------------------- tiles
// A step is written as matrix ops with, between two of them, a piece of the
// vector work that does not depend on the tile in flight: selection and hi/lo
// split of the tile before, decode of the next FP8 chunk.  A matrix op takes
// 16 cycles of one wave's issue and hides up to three independent vector ops
// (16.8 cycles alone; 18.4, 20.2 and 20.9 with one, two and three after it).
template <class D, int CHI>
struct TileOp;
template <int CHI>
struct TileOp<DF32, CHI> {
  static constexpr int NV = CHI / 16, NCH = CHI / 16;  // chunks of four 4-wide ops
  static constexpr int OPC = 4;                        // ops per chunk, slice and column group
  struct Operand { u32x4 w; };
  template <class F>
  __device__ __forceinline__ static void decode(const F& f, int c, int piece, Operand& x) {
    if (piece == 0) x.w = u32x4{f.w[4 * c], f.w[4 * c + 1], f.w[4 * c + 2], f.w[4 * c + 3]};
  }
  static constexpr int kPieces = 1;
  __device__ __forceinline__ static f4 op(const Operand& x, const u32x4 (&r)[NV], int c, int k, f4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.w[k]), __uint_as_float(r[c][k]), acc, 0, 0, 0);
  }
  // output tile j of a wave's tiles into its words, in kStages pieces
  struct Post { f4 v; };
  static constexpr int kStages = 4;
  template <bool RN, int MT>
  __device__ __forceinline__ static void post(int st, Post& p, bool bit, const f4& c0, const f4& c1, float psc,
                                              u32x4 (&o)[MT], int j) {
    float v = bit ? c1[st] : c0[st];
    if constexpr (RN) v *= psc;
    o[j][st] = __float_as_uint(v);
  }
  // exponent of the largest |x| of the walker's vector
  __device__ __forceinline__ static int row_exp(const u32x4 (&r)[NV]) {
    float mx = 0.f;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, fabsf(__uint_as_float(r[v][i])));
    mx = group_max(mx);
    return (mx > 0.f) ? __builtin_amdgcn_frexp_expf(mx) : 0;
  }
  static constexpr uint32_t kUnit = 0x3F800000u;  // first word of e_0
  // FP64 dot product of MT words of a row and of a column
  template <int MT>
  __device__ __forceinline__ static double dot(const u32x4 (&r)[MT], const u32x4 (&c)[MT]) {
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < MT; ++v)
#pragma unroll
      for (int i = 0; i < 4; ++i) s = fma((double)__uint_as_float(r[v][i]), (double)__uint_as_float(c[v][i]), s);
    return s;
  }
};
template <int CHI>
struct TileOp<DBF16, CHI> {
  static constexpr int NV = CHI / 16, NCH = CHI / 32;  // chunks of 32 features
  static constexpr int OPC = 2;                        // hi part, lo part
  struct Operand { bf16x8 x; };
  template <class F>
  __device__ __forceinline__ static void decode(const F& f, int c, int piece, Operand& x) {
    if (piece == 0) x.x = DBF16::template pack<CHI / 4>(f, c);
  }
  static constexpr int kPieces = 1;
  // words 2c and 2c + 1 of a vector: hi and lo parts of tiles 2c and 2c + 1
  __device__ __forceinline__ static f4 op(const Operand& x, const u32x4 (&r)[NV], int c, int k, f4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.x, __builtin_bit_cast(bf16x8, r[2 * c + k]), acc, 0, 0, 0);
  }
  struct Post { float a, b, d; uint32_t h; };
  static constexpr int kStages = 8;
  template <bool RN, int MT>
  __device__ __forceinline__ static void post(int st, Post& p, bool bit, const f4& c0, const f4& c1, float psc,
                                              u32x4 (&o)[MT], int j) {
    const int e = st / 4 * 2, c = j / 2, q = 2 * (j % 2) + st / 4;
    if (st % 4 == 0) {
      p.a = bit ? c1[e] : c0[e];
      p.b = bit ? c1[e + 1] : c0[e + 1];
      if constexpr (RN) {
        p.a *= psc;
        p.b *= psc;
      }
    } else if (st % 4 == 1) {
      p.h = pack_bf16x2(p.a, p.b);
      o[2 * c][q] = p.h;
      p.d = __uint_as_float(p.h << 16);
    } else if (st % 4 == 2) {
      p.a -= p.d;
      p.d = __uint_as_float(p.h & 0xffff0000u);
    } else {
      p.b -= p.d;
      o[2 * c + 1][q] = pack_bf16x2(p.a, p.b);
    }
  }
  // (from the hi parts: any power of two is exact, and every wave derives the
  // same one from the same bits)
  __device__ __forceinline__ static int row_exp(const u32x4 (&r)[NV]) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    us2 mx = {0, 0};
#pragma unroll
    for (int c = 0; c < NV / 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        mx = __builtin_elementwise_max(mx, __builtin_bit_cast(us2, r[2 * c][i] & 0x7fff7fffu));
    const float f = group_max(__uint_as_float((uint32_t)(mx[0] > mx[1] ? mx[0] : mx[1]) << 16));
    return (f > 0.f) ? __builtin_amdgcn_frexp_expf(f) : 0;
  }
  static constexpr uint32_t kUnit = 0x3F80u;
  template <int MT>
  __device__ __forceinline__ static double dot(const u32x4 (&r)[MT], const u32x4 (&c)[MT]) {
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < MT / 2; ++v)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int q = i / 2, sh = 16 * (1 - i % 2);  // low half first
        auto val = [&](const u32x4& h, const u32x4& l) {
          return __uint_as_float((h[q] << sh) & 0xffff0000u) + __uint_as_float((l[q] << sh) & 0xffff0000u);
        };
        s = fma((double)val(r[2 * v], r[2 * v + 1]), (double)val(c[2 * v], c[2 * v + 1]), s);
      }
    return s;
  }
};
template <int CHI>
struct TileOp<DFP8, CHI> : TileOp<DBF16, CHI> {
  // the 8 codes of chunk c decoded to BF16 values, one conversion (two codes) per piece
  static constexpr int kPieces = 4;
  struct Operand { u32x4 x; };
  template <class F>
  __device__ __forceinline__ static void decode(const F& f, int c, int piece, Operand& x) {
    const uint32_t w = f.w[2 * c + piece / 2];
    x.x[piece] = __builtin_bit_cast(uint32_t, piece % 2 ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, kFp8Scale, true)
                                                        : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, kFp8Scale, false));
  }
  __device__ __forceinline__ static f4 op(const Operand& x, const u32x4 (&r)[CHI / 16], int c, int k, f4 acc) {
    return TileOp<DBF16, CHI>::op({__builtin_bit_cast(bf16x8, x.x)}, r, c, k, acc);
  }
};

// element i of a table that is not written while the kernel runs, at a
// wave-uniform index: a scalar load
template <class V>
__device__ __forceinline__ V uniform_load(const V* p, long long i) {
  typedef const __attribute__((address_space(4))) V* cptr;
  return ((cptr)(uintptr_t)p)[i];
}

// a pointer that is the same in every lane, in scalar registers
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t u = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const char*)(uintptr_t)((uint64_t)hi << 32 | lo);
}

}  // namespace rttk
