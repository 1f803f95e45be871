// Learned multi-spin proposal on gfx950: a 3-layer 3x3 convolutional
// network (32 channels, SiLU, periodic padding) with a 1x1 head giving, per
// site, one centre logit and eight size logits.  A move flips the first k
// sites of a fixed spiral around a sampled centre; the Metropolis-Hastings
// ratio uses the exact proposal probability of the flipped set in both
// directions, so the chain samples |psi|^2 whatever the weights are.
//
// One block of 256 threads per configuration, one thread per lattice site
// (N <= 256).  Weights are read with uniform addresses (scalar loads);
// activations live in LDS as [channel][site].
#pragma once
#include "rtt_device.hpp"

namespace rttk {

constexpr int kNetC = 32;
constexpr int kNetParams = 19113;
// offsets of the flattened parameters: W1, b1, W2, b2, W3, b3, Wh, bh
constexpr int oW1 = 0, ob1 = 288, oW2 = 320, ob2 = 9536, oW3 = 9568, ob3 = 18784, oWh = 18816,
              obh = 19104;
// spiral (dx, dy) around the centre
__constant__ const int kSpiralDx[8] = {0, 1, 1, 0, -1, -1, -1, 0};
__constant__ const int kSpiralDy[8] = {0, 0, 1, 1, 1, 0, -1, -1};

__device__ __forceinline__ float silu_f(float a) { return a / (1.f + __expf(-a)); }
__device__ __forceinline__ float silu_grad(float a) {
  const float s = 1.f / (1.f + __expf(-a));
  return s * (1.f + a * (1.f - s));
}

struct NetGeo {
  int Lx, Ly, N;
  int nb[9];  // neighbour (y + ky - 1, x + kx - 1) of this thread's site, tap = 3 ky + kx
  __device__ void init(int lx, int ly) {
    Lx = lx; Ly = ly; N = lx * ly;
    const int i = threadIdx.x < N ? threadIdx.x : 0;
    const int x = i % lx, y = i / lx;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int ky = t / 3, kx = t % 3;
      nb[t] = ((y + ky - 1 + ly) % ly) * lx + (x + kx - 1 + lx) % lx;
    }
  }
};

// The first layer (one input channel) for this thread's site: acc[co] = b[co] + sum W[co][t] z(nb[t]).
__device__ __forceinline__ void conv_site(const float* __restrict__ W, const float* __restrict__ b, const float* z,
                                          const NetGeo& g, float (&acc)[kNetC]) {
#pragma unroll
  for (int co = 0; co < kNetC; ++co) acc[co] = b[co];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const float x = z[g.nb[t]];
#pragma unroll
    for (int co = 0; co < kNetC; ++co) acc[co] = fmaf(W[co * 9 + t], x, acc[co]);
  }
}

// ---------------------------------------------------------------- matrix-core forward
// The two 32 -> 32 channel 3x3 layers as implicit GEMMs on the BF16 matrix
// cores: out^T[co][site] = sum over taps t and input channels ci of
// W[co][ci][t] h[ci][nb(site, t)], one 16 (channels) x 16 (sites) tile per
// matrix op sequence, K = 32 input channels per tap.  The weights are BF16
// values already; each activation enters as three BF16 parts hi + mid + lo
// (their sum equals it to about 2^-26 relative, finer than FP32 rounding),
// so with FP32 accumulation the layer keeps FP32 accuracy.  Activations are
// kept in LDS site-major, [site][channel], one plane per part.
// Packed weights: [layer 2, 3][tap][co][ci] BF16, written from the
// inference copy by net_pack_kernel.
constexpr int kNetPacked = 2 * 9 * kNetC * kNetC;

__global__ void net_pack_kernel(const float* infer, uint16_t* wpk) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kNetPacked) return;
  const int layer = p / (9 * kNetC * kNetC), r = p % (9 * kNetC * kNetC);
  const int t = r / (kNetC * kNetC), co = (r / kNetC) % kNetC, ci = r % kNetC;
  const float w = infer[(layer == 0 ? oW2 : oW3) + (co * kNetC + ci) * 9 + t];
  wpk[p] = f32_to_bf16_rne(w);  // exact: the inference weights are BF16 values
}

__device__ __forceinline__ void split3_bf16(float x, uint16_t& h, uint16_t& m, uint16_t& l) {
  const __bf16 xh = (__bf16)x;
  const float r1 = x - (float)xh;
  const __bf16 xm = (__bf16)r1;
  const __bf16 xl = (__bf16)(r1 - (float)xm);
  h = __builtin_bit_cast(uint16_t, xh);
  m = __builtin_bit_cast(uint16_t, xm);
  l = __builtin_bit_cast(uint16_t, xl);
}

// sites padded to whole 16-site tiles
__host__ __device__ inline int net_padded(int N) { return (N + 15) / 16 * 16; }
// LDS (floats) of the matrix-core forward kernels: z[256], two activation
// buffers of three [NP][32] BF16 planes (the first later holds SiLU(a3) as
// [32][N] floats), o[9][N], then the log-probability area of the proposal
// kernels (lc[N] doubles, lk[8][N], reduction scratch, move, flip set)
__host__ __device__ inline size_t net_fwd_lds_bytes(int N) {
  return (size_t)(280 + 96 * net_padded(N) + 19 * N) * 4;
}

// One 32 -> 32 layer: input planes in (SiLU'd activations, split), output
// SiLU(a) either split into the planes out, or as FP32 [32][N] into h3.
__device__ __forceinline__ void net_conv_mfma(const uint16_t* __restrict__ wl, const float* __restrict__ bias,
                                              const uint16_t* in, uint16_t* out, float* h3, const NetGeo& g,
                                              int NP) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gq = lane >> 4, m = lane & 15;
  const int ct = wave >> 1;  // output channel tile of this wave
  const int N = g.N;
  bf16x8 wa[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
    wa[t] = *reinterpret_cast<const bf16x8*>(wl + ((size_t)t * kNetC + ct * 16 + m) * kNetC + 8 * gq);
  float bv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bv[i] = bias[ct * 16 + 4 * gq + i];
  const size_t plane = (size_t)NP * kNetC;
  for (int st = wave & 1; st < NP / 16; st += 2) {
    const int site = st * 16 + m;
    const int sc = site < N ? site : 0;
    const int x = sc % g.Lx, y = sc / g.Lx;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      int yy = y + t / 3 - 1, xx = x + t % 3 - 1;
      yy += yy < 0 ? g.Ly : 0;
      yy -= yy >= g.Ly ? g.Ly : 0;
      xx += xx < 0 ? g.Lx : 0;
      xx -= xx >= g.Lx ? g.Lx : 0;
      const uint16_t* row = in + (size_t)(yy * g.Lx + xx) * kNetC + 8 * gq;
      const bf16x8 bl = *reinterpret_cast<const bf16x8*>(row + 2 * plane);
      const bf16x8 bm = *reinterpret_cast<const bf16x8*>(row + plane);
      const bf16x8 bh = *reinterpret_cast<const bf16x8*>(row);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[t], bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[t], bm, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[t], bh, acc, 0, 0, 0);
    }
    if (site < N) {  // lane holds channels ct*16 + 4gq .. +3 of this site
      const int c0 = ct * 16 + 4 * gq;
      if (h3) {
#pragma unroll
        for (int i = 0; i < 4; ++i) h3[(c0 + i) * N + site] = silu_f(acc[i] + bv[i]);
      } else {
        uint16_t ph[4], pm[4], pl[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) split3_bf16(silu_f(acc[i] + bv[i]), ph[i], pm[i], pl[i]);
        uint16_t* o = out + (size_t)site * kNetC + c0;
        *reinterpret_cast<uint2*>(o) = make_uint2(ph[0] | (uint32_t)ph[1] << 16, ph[2] | (uint32_t)ph[3] << 16);
        *reinterpret_cast<uint2*>(o + plane) =
            make_uint2(pm[0] | (uint32_t)pm[1] << 16, pm[2] | (uint32_t)pm[3] << 16);
        *reinterpret_cast<uint2*>(o + 2 * plane) =
            make_uint2(pl[0] | (uint32_t)pl[1] << 16, pl[2] | (uint32_t)pl[3] << 16);
      }
    }
  }
}

// Forward pass of one configuration with the layers above (256 threads:
// layer 1 and the head one thread per site, the two middle layers on the
// matrix cores).  Returns o[9][N] in LDS.
__device__ inline float* net_forward_mfma(const float* __restrict__ P, const uint16_t* __restrict__ wpk,
                                          const uint64_t* spins, const NetGeo& g, float* lds) {
  const int N = g.N, i = threadIdx.x, NP = net_padded(N);
  const bool act = i < N;
  float* z = lds;
  uint16_t* S0 = reinterpret_cast<uint16_t*>(lds + 256);
  uint16_t* S1 = S0 + 3 * NP * kNetC;
  float* H3 = reinterpret_cast<float*>(S0);  // S0 is free once layer 2 has run
  float* o = reinterpret_cast<float*>(S1 + 3 * NP * kNetC);
  if (act) z[i] = 1.f - 2.f * (float)spin_bit(spins, i);
  __syncthreads();
  if (act) {
    float acc[kNetC];
    conv_site(P + oW1, P + ob1, z, g, acc);
    const size_t plane = (size_t)NP * kNetC;
#pragma unroll
    for (int c = 0; c < kNetC; c += 2) {
      uint16_t h0, m0, l0, h1, m1, l1;
      split3_bf16(silu_f(acc[c]), h0, m0, l0);
      split3_bf16(silu_f(acc[c + 1]), h1, m1, l1);
      uint32_t* row = reinterpret_cast<uint32_t*>(S0 + (size_t)i * kNetC + c);
      row[0] = h0 | (uint32_t)h1 << 16;
      row[plane / 2] = m0 | (uint32_t)m1 << 16;
      row[plane] = l0 | (uint32_t)l1 << 16;
    }
  }
  __syncthreads();
  net_conv_mfma(wpk, P + ob2, S0, S1, nullptr, g, NP);
  __syncthreads();
  net_conv_mfma(wpk + 9 * kNetC * kNetC, P + ob3, S1, nullptr, H3, g, NP);
  __syncthreads();
  if (act) {
    float h[kNetC];
#pragma unroll
    for (int c = 0; c < kNetC; ++c) h[c] = H3[c * N + i];
    for (int k = 0; k < 9; ++k) {
      float s = P[obh + k];
#pragma unroll
      for (int c = 0; c < kNetC; ++c) s = fmaf(P[oWh + k * kNetC + c], h[c], s);
      o[k * N + i] = s;
    }
  }
  __syncthreads();
  return o;
}

// block-wide reductions (256 threads)
__device__ inline double block_sum_d(double x, double* sh) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  const double r = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return r;
}
__device__ inline float block_max_f(float x, float* sh) {
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
  __syncthreads();
  const float r = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  __syncthreads();
  return r;
}

// log-softmax of the centre logits over sites (block) and of this thread's
// eight size logits; writes lc[i] (log p(c = i)) and lk[8][i] into LDS.
__device__ inline void net_logprobs(const float* o, const NetGeo& g, double* lc, float* lk, double* shd,
                                    float* shf) {
  const int N = g.N, i = threadIdx.x;
  const bool act = i < N;
  const float m = block_max_f(act ? o[i] : -INFINITY, shf);
  const double se = block_sum_d(act ? exp((double)o[i] - (double)m) : 0.0, shd);
  const double lse = (double)m + log(se);
  if (act) {
    lc[i] = (double)o[i] - lse;
    float mk = -INFINITY;
    for (int k = 0; k < 8; ++k) mk = fmaxf(mk, o[(k + 1) * N + i]);
    double s = 0.0;
    for (int k = 0; k < 8; ++k) s += exp((double)o[(k + 1) * N + i] - (double)mk);
    const double l = (double)mk + log(s);
    for (int k = 0; k < 8; ++k) lk[k * N + i] = (float)((double)o[(k + 1) * N + i] - l);
  }
  __syncthreads();
}

__device__ __forceinline__ int spiral_site(int c, int m, int Lx, int Ly) {
  const int x = c % Lx, y = c / Lx;
  return ((y + kSpiralDy[m] + Ly) % Ly) * Lx + (x + kSpiralDx[m] + Lx) % Lx;
}

// q(S|s) for the flip set S of move (c, k): sum of p(c') p(k|c') over the
// centres c' whose k-site spiral equals S (sets of different sizes differ).
__device__ inline double net_set_prob(const double* lc, const float* lk, const NetGeo& g, int c, int k,
                                      const uint64_t* target, double* shd) {
  const int i = threadIdx.x;
  double p = 0.0;
  if (i < g.N) {
    bool same = true;
    for (int m = 0; m < k; ++m) {
      const int s = spiral_site(i, m, g.Lx, g.Ly);
      same &= ((target[s >> 6] >> (s & 63)) & 1ull) != 0ull;
    }
    if (same) p = exp(lc[i] + (double)lk[(k - 1) * g.N + i]);
  }
  return block_sum_d(p, shd);
}

struct NetMoveArgs {
  const float* P;          // inference weights
  const uint16_t* wpk;     // the middle layers' weights packed for the matrix cores
  int Lx, Ly, nw, W;
  const uint64_t* spins;   // [W][nw] current
  uint64_t* prop;          // [W][nw] proposed (written by propose)
  int* moves;              // [W] c | k << 16
  double* lqf;             // [W] log q(S|s)
  double* lqr;             // [W] log q(S|s')
  uint64_t seed, rstream, step;
  float* out;              // [W][9][N] head outputs (forward only) or null
  uint64_t* before;        // [W][nw] copy of the state the move was proposed at, or null
};

// propose: forward at s, sample (c, k), write s' and log q(S|s)
__global__ void __launch_bounds__(256) net_propose_kernel(NetMoveArgs a) {
  extern __shared__ __align__(16) float lds[];
  NetGeo g;
  g.init(a.Lx, a.Ly);
  const int w = blockIdx.x, N = g.N;
  const uint64_t* sw = a.spins + (size_t)w * a.nw;
  float* o = net_forward_mfma(a.P, a.wpk, sw, g, lds);
  double* lc = reinterpret_cast<double*>(o + 9 * N + (N & 1));
  float* lk = reinterpret_cast<float*>(lc + N);
  double* shd = reinterpret_cast<double*>(lk + 8 * N + ((8 * N) & 1));
  float* shf = reinterpret_cast<float*>(shd + 4);
  int* mv = reinterpret_cast<int*>(shf + 4);
  uint64_t* tgt = reinterpret_cast<uint64_t*>(mv + 2);
  net_logprobs(o, g, lc, lk, shd, shf);
  // inverse-CDF draw of the centre: inclusive prefix sums of p(c = i) over
  // the sites (FP64 block scan in site order), c = the first site whose sum
  // exceeds uc (the last site if none does)
  {
    const int i = threadIdx.x, lane = i & 63, wv = i >> 6;
    const double uc = philox_uniform(a.seed, a.rstream, (uint64_t)w, a.step, (1ull << 32) + 0);
    double cum = i < N ? exp(lc[i]) : 0.0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double y = __shfl_up(cum, o);
      if (lane >= o) cum += y;
    }
    if (lane == 63) shd[wv] = cum;
    __syncthreads();
    for (int q = 0; q < wv; ++q) cum += shd[q];
    int cand = (i < N && cum > uc) ? i : N - 1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cand = min(cand, __shfl_xor(cand, o));
    int* shi = reinterpret_cast<int*>(shf);
    __syncthreads();
    if (lane == 0) shi[wv] = cand;
    __syncthreads();
    if (i == 0) mv[0] = min(min(shi[0], shi[1]), min(shi[2], shi[3]));
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double uk = philox_uniform(a.seed, a.rstream, (uint64_t)w, a.step, (1ull << 32) + 1);
    const int c = mv[0];
    double cum = 0.0;
    int k = 8;
    for (int m = 0; m < 8; ++m) {
      cum += exp((double)lk[m * N + c]);
      if (cum > uk) { k = m + 1; break; }
    }
    mv[0] = c;
    mv[1] = k;
    for (int q = 0; q < a.nw; ++q) tgt[q] = 0ull;
    for (int m = 0; m < k; ++m) {
      const int s = spiral_site(c, m, a.Lx, a.Ly);
      tgt[s >> 6] |= 1ull << (s & 63);
    }
  }
  __syncthreads();
  const int c = mv[0], k = mv[1];
  const double q = net_set_prob(lc, lk, g, c, k, tgt, shd);
  if (threadIdx.x == 0) {
    a.moves[w] = c | (k << 16);
    a.lqf[w] = log(q);
  }
  if (threadIdx.x < a.nw) {
    a.prop[(size_t)w * a.nw + threadIdx.x] = sw[threadIdx.x] ^ tgt[threadIdx.x];
    if (a.before) a.before[(size_t)w * a.nw + threadIdx.x] = sw[threadIdx.x];
  }
}

// reverse: forward at s', log q(S|s') for the same set
__global__ void __launch_bounds__(256) net_reverse_kernel(NetMoveArgs a) {
  extern __shared__ __align__(16) float lds[];
  NetGeo g;
  g.init(a.Lx, a.Ly);
  const int w = blockIdx.x, N = g.N;
  float* o = net_forward_mfma(a.P, a.wpk, a.prop + (size_t)w * a.nw, g, lds);
  double* lc = reinterpret_cast<double*>(o + 9 * N + (N & 1));
  float* lk = reinterpret_cast<float*>(lc + N);
  double* shd = reinterpret_cast<double*>(lk + 8 * N + ((8 * N) & 1));
  float* shf = reinterpret_cast<float*>(shd + 4);
  int* mv = reinterpret_cast<int*>(shf + 4);
  uint64_t* tgt = reinterpret_cast<uint64_t*>(mv + 2);
  net_logprobs(o, g, lc, lk, shd, shf);
  const int c = a.moves[w] & 0xffff, k = a.moves[w] >> 16;
  if (threadIdx.x == 0) {
    for (int q = 0; q < a.nw; ++q) tgt[q] = 0ull;
    for (int m = 0; m < k; ++m) {
      const int s = spiral_site(c, m, a.Lx, a.Ly);
      tgt[s >> 6] |= 1ull << (s & 63);
    }
  }
  __syncthreads();
  const double q = net_set_prob(lc, lk, g, c, k, tgt, shd);
  if (threadIdx.x == 0) a.lqr[w] = log(q);
}

// forward only: head outputs to global memory
__global__ void __launch_bounds__(256) net_forward_kernel(NetMoveArgs a) {
  extern __shared__ __align__(16) float lds[];
  NetGeo g;
  g.init(a.Lx, a.Ly);
  const int w = blockIdx.x, N = g.N;
  const float* o = net_forward_mfma(a.P, a.wpk, a.spins + (size_t)w * a.nw, g, lds);
  for (int i = threadIdx.x; i < 9 * N; i += 256) a.out[(size_t)w * 9 * N + i] = o[i];
}

// acceptance (one thread per walker): u < |psi'/psi|^2 q(S|s') / q(S|s)
struct NetAcceptArgs {
  int W, nw;
  uint64_t* spins; const uint64_t* prop;
  double* logabs; int8_t* sign;
  const double* la_new; const int8_t* sg_new; const int32_t* st_new;
  const double* lqf; const double* lqr;
  const int* moves; float* accept_prob;
  uint32_t* accepts; int32_t* status;
  uint64_t seed, rstream, step;
};
__global__ void net_accept_kernel(NetAcceptArgs a) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= a.W) return;
  const bool ok_old = isfinite(a.logabs[w]) && a.sign[w] != 0;
  const bool ok_new = a.st_new[w] == 0;
  double A = 0.0;
  if (ok_old && ok_new) A = exp(2.0 * (a.la_new[w] - a.logabs[w]) + a.lqr[w] - a.lqf[w]);
  const double u = philox_uniform(a.seed, a.rstream, (uint64_t)w, a.step, (1ull << 32) + 2);
  const bool acc = ok_old && ok_new && u < A;
  if (a.accept_prob) a.accept_prob[w] = (float)fmin(1.0, A);
  if (acc) {
    for (int q = 0; q < a.nw; ++q) a.spins[(size_t)w * a.nw + q] = a.prop[(size_t)w * a.nw + q];
    a.logabs[w] = a.la_new[w];
    a.sign[w] = a.sg_new[w];
    if (a.accepts) a.accepts[w] += 1;
  }
  if (a.status) a.status[w] = ok_old ? 0 : -5;
}

// ---------------------------------------------------------------- training
struct NetGradArgs {
  const float* P;          // weights the forward pass uses
  int Lx, Ly, nw, B;
  const uint64_t* spins;   // [B][nw] states s_b
  const int* moves;        // [B] c | k << 16 sampled at s_b
  const float* accept_prob;// [B]
  const double* baseline;  // device scalar
  float* partial;          // [blocks][kNetParams] partial gradients
};

// Gradient of sum_b coef_b log q(c_b, k_b | s_b), coef_b = -(a_b k_b - baseline)
// / B, on the FP32 matrix cores.  A block takes samples b, b + gridDim, ... and
// sums their weight gradients; one partial gradient per block then goes to
// memory (a gradient per sample was 313 MB written and read back at 4096
// samples).
//   conv layers and their transposes: out[ch][site], 16 x 16 tiles, K = 9 taps
//     x 32 channels;
//   weight gradients: dW[co][ci][t] = sum_i da[co][i] h[ci][nb(i, t)], wave
//     (co tile, ci tile), nine tap tiles, K = sites;
//   head and first layer: their 9 outputs or taps padded to 16.
// Activations are [site][32] floats in LDS, the 16-byte chunks of a row swizzled
// by (site / 2) % 8 so that 16 consecutive sites read one chunk conflict-free.
// Buffers: X0 a1 -> da1; X1 h1 -> a3 -> da3; X2 a2 -> da2; X3 h2 -> h1.
// Matrix ops of 4096 samples at 10x10 take 330 us of all 1024 SIMDs; measured
// 0.99 ms (one thread per site or weight, a gradient per sample: 3.5 ms with
// the sum over samples), the rest being layer weights, LDS reads, barriers and
// scratch: the 72 weights a lane holds in a layer and the 72 sums of a sample
// leave no room for the block's sums, which spill (796 bytes a lane).
__device__ __forceinline__ int gidx(int site, int ch) {
  return site * kNetC + ((((ch >> 2) ^ (site >> 1)) & 7) << 2) + (ch & 3);
}
__device__ __forceinline__ f4 gread4(const float* X, int site, int ch) {
  return *reinterpret_cast<const f4*>(X + gidx(site, ch));
}
__device__ __forceinline__ void gwrite4(float* X, int site, int ch, f4 v) {
  *reinterpret_cast<f4*>(X + gidx(site, ch)) = v;
}
__device__ __forceinline__ f4 mfma_f32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LDS (floats): z[256], X0..X3, o[9][N], the log-probabilities and scratch of
// net_logprobs, the neighbour table [9][256] (bytes)
__host__ __device__ inline size_t net_grad_lds_bytes(int N) { return (size_t)(280 + 147 * N + 9 * 64) * 4; }

// One 32 -> 32 layer over the block's sites: fin(site, ch, v) takes channels ch
// .. ch + 3 of a site.  wt[t][e]: this lane's weights of tap t, input channel
// 8 g + e; tap t reads the site nb[flip ? 8 - t : t].
template <class F>
__device__ __forceinline__ void net_grad_conv(const float (&wt)[9][8], const float* X, const uint8_t* nbt, int N,
                                              bool flip, F&& fin) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, m = lane & 15, ct = wave & 1;
  for (int st = wave >> 1; st < (N + 15) / 16; st += 2) {
    const int site = st * 16 + m, sc = site < N ? site : 0;
    // one sum per row of taps: shorter chains, and less rounding than one of 288
    f4 acc[3];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int nb = nbt[(flip ? 8 - t : t) * 256 + sc];
      const f4 lo = gread4(X, nb, 8 * g), hi = gread4(X, nb, 8 * g + 4);
      f4& x = acc[t / 3];
      if (t % 3 == 0) x = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) x = mfma_f32(wt[t][e], lo[e], x);
#pragma unroll
      for (int e = 0; e < 4; ++e) x = mfma_f32(wt[t][4 + e], hi[e], x);
    }
    if (site < N) fin(site, ct * 16 + 4 * g, (acc[0] + acc[1]) + acc[2]);
  }
}

// dW += da^T h over the sites for this wave's (co tile, ci tile) and all taps;
// db += da (co of this lane).  A sample is summed by itself and then added: a
// chain over all of a block's samples would round more than a sum per sample.
__device__ __forceinline__ void net_grad_weights(const float* DA, const float* H, const uint8_t* nbt, int N, f4 (&dW)[9],
                                                 float& db) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, m = lane & 15, co = (wave & 1) * 16 + m, ci = (wave >> 1) * 16 + m;
  f4 w[9];
  float b = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) w[t] = f4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < N; s += 4) {
    const int site = s + g, sc = site < N ? site : 0;
    float a = DA[gidx(sc, co)];
    a = site < N ? a : 0.f;
    b += a;
#pragma unroll
    for (int t = 0; t < 9; ++t) w[t] = mfma_f32(a, H[gidx(nbt[t * 256 + sc], ci)], w[t]);
  }
  db += b;
#pragma unroll
  for (int t = 0; t < 9; ++t) dW[t] += w[t];
}

__global__ void __launch_bounds__(256, 2) net_grad_kernel(NetGradArgs a) {
  extern __shared__ __align__(16) float lds[];
  NetGeo geo;
  geo.Lx = a.Lx; geo.Ly = a.Ly; geo.N = a.Lx * a.Ly;
  const int N = geo.N, i = threadIdx.x;
  const bool act = i < N;
  const int lane = i & 63, wave = i >> 6, g = lane >> 4, m = lane & 15;
  float* z = lds;
  float* X0 = z + 256;
  float* X1 = X0 + kNetC * N;
  float* X2 = X1 + kNetC * N;
  float* X3 = X2 + kNetC * N;
  float* o = X3 + kNetC * N;
  double* lc = reinterpret_cast<double*>(o + 9 * N + (N & 1));
  float* lk = reinterpret_cast<float*>(lc + N);
  double* shd = reinterpret_cast<double*>(lk + 8 * N + ((8 * N) & 1));
  float* shf = reinterpret_cast<float*>(shd + 4);
  uint8_t* nbt = reinterpret_cast<uint8_t*>(lds + 280 + 147 * N);
  for (int p = i; p < 9 * 256; p += 256) {
    const int t = p / 256, s = p % 256 < N ? p % 256 : 0, x = s % a.Lx, y = s / a.Lx;
    nbt[p] = (uint8_t)(((y + t / 3 - 1 + a.Ly) % a.Ly) * a.Lx + (x + t % 3 - 1 + a.Lx) % a.Lx);
  }
  const float* __restrict__ P = a.P;
  // elementwise work: this thread's four channels of every 32nd site
  const int ec = 4 * (i & 7), es = i >> 3;
  // sums over the block's samples
  f4 dW3[9], dW2[9], dW1 = {0.f, 0.f, 0.f, 0.f}, dWh = {0.f, 0.f, 0.f, 0.f};
  float db3 = 0.f, db2 = 0.f, db1 = 0.f, dbh = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) { dW3[t] = f4{0.f, 0.f, 0.f, 0.f}; dW2[t] = f4{0.f, 0.f, 0.f, 0.f}; }
  const int ct = wave & 1;
  // this lane's weights of a layer (row 16 ct + m of the product), forward or transposed
  auto weights = [&](int oW, bool tr, float (&wt)[9][8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int co = tr ? 8 * g + e : 16 * ct + m, ci = tr ? 16 * ct + m : 8 * g + e;
#pragma unroll
      for (int t = 0; t < 9; ++t) wt[t][e] = P[oW + (co * kNetC + ci) * 9 + t];
    }
  };
  for (int b = blockIdx.x; b < a.B; b += gridDim.x) {
    const uint64_t* sw = a.spins + (size_t)b * a.nw;
    __syncthreads();  // the last sample's buffers are free
    if (act) z[i] = 1.f - 2.f * (float)spin_bit(sw, i);
    __syncthreads();
    // layer 1: a1 -> X0, h1 -> X1
    for (int s = es; s < N; s += 32) {
      f4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = P[ob1 + ec + q];
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const float x = z[nbt[t * 256 + s]];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fmaf(P[oW1 + (ec + q) * 9 + t], x, v[q]);
      }
      gwrite4(X0, s, ec, v);
      gwrite4(X1, s, ec, f4{silu_f(v[0]), silu_f(v[1]), silu_f(v[2]), silu_f(v[3])});
    }
    __syncthreads();
    // layer 2: a2 -> X2, h2 -> X3
    {
      float wt[9][8];
      weights(oW2, false, wt);
      net_grad_conv(wt, X1, nbt, N, false, [&](int s, int ch, f4 v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] += P[ob2 + ch + q];
        gwrite4(X2, s, ch, v);
        gwrite4(X3, s, ch, f4{silu_f(v[0]), silu_f(v[1]), silu_f(v[2]), silu_f(v[3])});
      });
    }
    __syncthreads();
    // layer 3: a3 -> X1
    {
      float wt[9][8];
      weights(oW3, false, wt);
      net_grad_conv(wt, X3, nbt, N, false, [&](int s, int ch, f4 v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] += P[ob3 + ch + q];
        gwrite4(X1, s, ch, v);
      });
    }
    __syncthreads();
    // head: o[k][site], k on the tile's rows
    {
      float wh[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) wh[e] = m < 9 ? P[oWh + m * kNetC + 8 * g + e] : 0.f;
      for (int st = wave; st < (N + 15) / 16; st += 4) {
        const int site = st * 16 + m, sc = site < N ? site : 0;
        const f4 lo = gread4(X1, sc, 8 * g), hi = gread4(X1, sc, 8 * g + 4);
        f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = mfma_f32(wh[e], silu_f(e < 4 ? lo[e & 3] : hi[e & 3]), acc);
        if (site < N)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (4 * g + q < 9) o[(4 * g + q) * N + site] = acc[q] + P[obh + 4 * g + q];
      }
    }
    __syncthreads();
    net_logprobs(o, geo, lc, lk, shd, shf);
    const int c = a.moves[b] & 0xffff, k = a.moves[b] >> 16;
    const double coef = -((double)a.accept_prob[b] * k - *a.baseline) / a.B;
    // d loss / d o, written over o: channel 0 at every site, size channels at c
    if (act) {
      o[i] = (float)(coef * ((i == c ? 1.0 : 0.0) - exp(lc[i])));
      for (int q = 0; q < 8; ++q)
        o[(q + 1) * N + i] = (i == c) ? (float)(coef * ((q + 1 == k ? 1.0 : 0.0) - exp((double)lk[q * N + i]))) : 0.f;
    }
    __syncthreads();
    // head: dWh[k][ch] += sum_i do[k][i] h3[ch][i] (waves 0 and 1: channel tiles)
    if (wave < 2) {
      f4 w = {0.f, 0.f, 0.f, 0.f};
      float bsum = 0.f;
      for (int s = 0; s < N; s += 4) {
        const int site = s + g, sc = site < N ? site : 0;
        const float d = m < 9 && site < N ? o[m * N + sc] : 0.f;
        bsum += d;
        w = mfma_f32(d, silu_f(X1[gidx(sc, 16 * wave + m)]), w);
      }
      dbh += bsum;
      dWh += w;
    }
    __syncthreads();
    // da3 = (Wh^T do) SiLU'(a3) -> X1
    for (int s = es; s < N; s += 32) {
      f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q9 = 0; q9 < 9; ++q9) {
        const float d = o[q9 * N + s];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fmaf(P[oWh + q9 * kNetC + ec + q], d, v[q]);
      }
      const f4 a3 = gread4(X1, s, ec);
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] *= silu_grad(a3[q]);
      gwrite4(X1, s, ec, v);
    }
    __syncthreads();
    // layer 3: dW3 from da3 and h2; da2 = (W3^T da3) SiLU'(a2) -> X2
    net_grad_weights(X1, X3, nbt, N, dW3, db3);
    {
      float wt[9][8];
      weights(oW3, true, wt);
      net_grad_conv(wt, X1, nbt, N, true, [&](int s, int ch, f4 v) {
        const f4 a2 = gread4(X2, s, ch);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] *= silu_grad(a2[q]);
        gwrite4(X2, s, ch, v);
      });
    }
    __syncthreads();
    // h1 -> X3
    for (int s = es; s < N; s += 32) {
      const f4 v = gread4(X0, s, ec);
      gwrite4(X3, s, ec, f4{silu_f(v[0]), silu_f(v[1]), silu_f(v[2]), silu_f(v[3])});
    }
    __syncthreads();
    // layer 2: dW2 from da2 and h1; da1 = (W2^T da2) SiLU'(a1) -> X0
    net_grad_weights(X2, X3, nbt, N, dW2, db2);
    {
      float wt[9][8];
      weights(oW2, true, wt);
      net_grad_conv(wt, X2, nbt, N, true, [&](int s, int ch, f4 v) {
        const f4 a1 = gread4(X0, s, ch);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] *= silu_grad(a1[q]);
        gwrite4(X0, s, ch, v);
      });
    }
    __syncthreads();
    // layer 1: dW1[co][t] += sum_i da1[co][i] z[nb(i, t)] (waves 0 and 1), taps on the tile's columns
    if (wave < 2) {
      f4 w = {0.f, 0.f, 0.f, 0.f};
      float bsum = 0.f;
      for (int s = 0; s < N; s += 4) {
        const int site = s + g, sc = site < N ? site : 0;
        float d = X0[gidx(sc, 16 * wave + m)];
        d = site < N ? d : 0.f;
        bsum += d;
        w = mfma_f32(d, m < 9 ? z[nbt[m * 256 + sc]] : 0.f, w);
      }
      db1 += bsum;
      dW1 += w;
    }
  }
  // the block's partial gradient: lane (g, m) holds rows 4 g + q and column m of its tiles
  float* out = a.partial + (size_t)blockIdx.x * kNetParams;
  db3 = group_sum(db3);
  db2 = group_sum(db2);
  db1 = group_sum(db1);
  dbh = group_sum(dbh);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int co = ct * 16 + 4 * g + q, ci = (wave >> 1) * 16 + m;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      out[oW3 + (co * kNetC + ci) * 9 + t] = dW3[t][q];
      out[oW2 + (co * kNetC + ci) * 9 + t] = dW2[t][q];
    }
    if (wave < 2) {
      if (m < 9) out[oW1 + (16 * wave + 4 * g + q) * 9 + m] = dW1[q];
      if (4 * g + q < 9) out[oWh + (4 * g + q) * kNetC + 16 * wave + m] = dWh[q];
    }
  }
  if (g == 0 && wave < 2) {
    out[ob3 + 16 * wave + m] = db3;
    out[ob2 + 16 * wave + m] = db2;
    out[ob1 + 16 * wave + m] = db1;
    if (wave == 0 && m < 9) out[obh + m] = dbh;
  }
}

// Sum over the blocks' partial gradients in two fixed-order stages: slice y of
// S adds its share, then net_reduce_kernel adds the S slices.
__global__ void net_reduce_slices_kernel(const float* partial, int B, int S, float* out) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
  if (p >= kNetParams) return;
  const int b0 = (int)((long long)B * y / S), b1 = (int)((long long)B * (y + 1) / S);
  float s = 0.f;
  for (int b = b0; b < b1; ++b) s += partial[(size_t)b * kNetParams + p];
  out[(size_t)y * kNetParams + p] = s;
}

// grad[p] = sum_b partial[b][p] (fixed order); baseline <- 0.9 baseline + 0.1 mean(a k)
__global__ void net_reduce_kernel(const float* partial, int B, float* grad) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kNetParams) return;
  float s = 0.f;
  for (int b = 0; b < B; ++b) s += partial[(size_t)b * kNetParams + p];
  grad[p] = s;
}
__global__ void net_baseline_kernel(const float* accept_prob, const int* moves, int B, double* baseline) {
  __shared__ double sh[4];
  double s = 0.0;
  for (int b = threadIdx.x; b < B; b += 256) s += (double)accept_prob[b] * (moves[b] >> 16);
  s = block_sum_d(s, sh);
  if (threadIdx.x == 0) *baseline = 0.9 * *baseline + 0.1 * (s / B);
}

// Adam on the FP32 master weights; the inference copy is rounded to BF16
__global__ void net_adam_kernel(float* master, float* infer, float* m, float* v, const float* grad,
                                float lr, float b1, float b2, float eps, int t) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kNetParams) return;
  const float gp = grad[p];
  const float mp = b1 * m[p] + (1.f - b1) * gp;
  const float vp = b2 * v[p] + (1.f - b2) * gp * gp;
  m[p] = mp;
  v[p] = vp;
  const float mh = mp / (1.f - powf(b1, (float)t));
  const float vh = vp / (1.f - powf(b2, (float)t));
  const float w = master[p] - lr * mh / (sqrtf(vh) + eps);
  master[p] = w;
  infer[p] = bf16_to_f32(f32_to_bf16_rne(w));
}

}  // namespace rttk
