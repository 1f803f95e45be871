// Estimator kernels (gfx950), independent of the core type.
//
//  combine_kernel  meets forward and backward vectors at the cut: amplitude,
//                  every single-flip ratio, linear-combination sums and the
//                  TFIM local energy, all in FP64.
//  reduce_kernel   compensated FP64 sums of local energies.
#pragma once
#include "rtt_kernels.hpp"

namespace rttk {

// ============================================================================
// combine kernel (one wave per walker)
// ============================================================================
struct CombineArgs {
  const float* u; const int32_t* ue;  // forward  [T][ng][W][nsf][chi], [T][ng][W][nsf]
  const float* v; const int32_t* ve;  // backward [T][ng][W][nsb][chi], [T][ng][W][nsb]
  int nsf, nsb, chi, T, W, N, nw, ng;
  const int32_t* fslot;               // [N] forward slot of spin j in its group (0 = base)
  const int32_t* bslot;               // [N] backward slot of spin j in its group (0 = base)
  const int32_t* grp;                 // [N] row group of spin j
  const double* coeffs;               // [T]
  const uint64_t* spins;
  const int2* bonds; int nbonds; double J, h;
  double* logabs; int8_t* sign; double* logratio; int8_t* rsign; double* eloc; int32_t* status;
};

// value = mant * 2^ex with |mant| in [0.5, 1) (mant = 0 for zero) of the
// combined amplitude whose forward row is slot fs and backward row slot bs
// of row group gi.  Sixteen lanes (c16 = lane % 16) share one dot product:
// each reads every 16th float4 of the two rows (coalesced 256-byte runs per
// row), FP64 partial sums meet by butterfly; all sixteen lanes return it.
__device__ inline void combined_value(const CombineArgs& a, int w, int gi, int fs, int bs, int c16,
                                      double& mant, int& ex) {
  double ms[kMaxTerms];
  int es[kMaxTerms];
  int emax = INT_MIN;
  for (int t = 0; t < a.T; ++t) {
    const size_t ty = (size_t)t * a.ng + gi;
    const float* pu = a.u + ((ty * a.W + w) * a.nsf + fs) * a.chi;
    const float* pv = a.v + ((ty * a.W + w) * a.nsb + bs) * a.chi;
    double d = 0.0;
    for (int f = 4 * c16; f < a.chi; f += 64) {
      const float4 x = *reinterpret_cast<const float4*>(pu + f);
      const float4 y = *reinterpret_cast<const float4*>(pv + f);
      d = fma((double)x.x, (double)y.x, d);
      d = fma((double)x.y, (double)y.y, d);
      d = fma((double)x.z, (double)y.z, d);
      d = fma((double)x.w, (double)y.w, d);
    }
    d += __shfl_xor(d, 8);
    d += __shfl_xor(d, 4);
    d += __shfl_xor(d, 2);
    d += __shfl_xor(d, 1);
    int ed = 0;
    const double md = frexp(d, &ed);
    ms[t] = a.coeffs[t] * md;
    es[t] = a.ue[(ty * a.W + w) * a.nsf + fs] + a.ve[(ty * a.W + w) * a.nsb + bs] + ed;
    if (ms[t] != 0.0 && es[t] > emax) emax = es[t];
  }
  if (emax == INT_MIN) { mant = 0.0; ex = 0; return; }
  double S = 0.0;
  for (int t = 0; t < a.T; ++t)
    if (ms[t] != 0.0) S += ldexp(ms[t], es[t] - emax);
  int eS = 0;
  mant = frexp(S, &eS);
  ex = emax + eS;
}

__device__ inline double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// One wave per walker; the wave's four 16-lane groups take four spins at a
// time.  Writes log|psi|, sign, status, every log|r_j| and sign, and E_loc.
__device__ __forceinline__ void combine_body(const CombineArgs& a, int bx) {
  const int lane = threadIdx.x & 63;
  const int q = lane >> 4, c16 = lane & 15;
  const int w = bx * 4 + (threadIdx.x >> 6);
  if (w >= a.W) return;
  const double LN2 = 0.69314718055994530942;
  double m0; int e0;
  combined_value(a, w, 0, 0, 0, c16, m0, e0);
  const bool ok = (m0 != 0.0) && isfinite(m0);
  const double lab0 = ok ? log(fabs(m0)) + e0 * LN2 : NAN;
  if (lane == 0) {
    if (a.logabs) a.logabs[w] = lab0;
    if (a.sign) a.sign[w] = ok ? (m0 > 0 ? 1 : -1) : 0;
    if (a.status) a.status[w] = ok ? 0 : -5;
  }
  double rsum = 0.0;
  for (int j0 = 0; j0 < a.N; j0 += 4) {
    const bool valid = j0 + q < a.N;
    const int j = valid ? j0 + q : a.N - 1;  // every group takes part in its butterfly
    const int fs = a.fslot[j], bs = a.bslot[j];
    double lr = NAN, r = NAN;
    int8_t sg = 0;
    if (ok) {
      if (fs == 0 && bs == 0) {  // spin read by no position: r_j = 1 exactly
        lr = 0.0; sg = 1; r = 1.0;
      } else {
        double mj; int ej;
        combined_value(a, w, a.grp[j], fs, bs, c16, mj, ej);
        if (mj == 0.0) { lr = -INFINITY; sg = 1; r = 0.0; }
        else {
          // the ratio from the mantissa quotient and the exponent difference
          // (no logarithms unless log-ratios are asked for)
          const double qm = fabs(mj) / fabs(m0);
          sg = ((mj > 0) == (m0 > 0)) ? 1 : -1;
          r = sg * ldexp(qm, ej - e0);
          if (a.logratio) lr = log(qm) + (double)(ej - e0) * LN2;
        }
      }
    }
    if (valid && c16 == 0) {
      if (a.logratio) a.logratio[(size_t)w * a.N + j] = lr;
      if (a.rsign) a.rsign[(size_t)w * a.N + j] = sg;
      rsum += ok ? r : 0.0;
    }
  }
  if (a.eloc) {
    const uint64_t* sw = a.spins + (size_t)w * a.nw;
    double diag = 0.0;
    for (int b = lane; b < a.nbonds; b += 64) {
      const int2 bd = a.bonds[b];
      diag += (spin_bit(sw, bd.x) ^ spin_bit(sw, bd.y)) ? -1.0 : 1.0;
    }
    diag = wave_sum(diag);
    rsum = wave_sum(rsum);
    if (lane == 0) a.eloc[w] = ok ? a.J * diag - a.h * rsum : NAN;
  }
}

__global__ void __launch_bounds__(256) combine_kernel(CombineArgs a) { combine_body(a, blockIdx.x); }

// ============================================================================
// compensated reduction
// ============================================================================
__device__ __forceinline__ void neumaier_add(double& s, double& c, double x) {
  const double t = s + x;
  c += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
  s = t;
}
__device__ __forceinline__ void neumaier_merge(double& s, double& c, double s2, double c2) {
  neumaier_add(s, c, s2);
  c += c2;
}

__device__ __forceinline__ void reduce_body(int n, const double* x, double* out) {
  __shared__ double sh[4][256];
  double s1 = 0, c1 = 0, s2 = 0, c2 = 0, cnt = 0;
  for (int i = threadIdx.x; i < n; i += 256) {
    const double v = x[i];
    if (!isfinite(v)) continue;
    neumaier_add(s1, c1, v);
    neumaier_add(s2, c2, v * v);
    cnt += 1.0;
  }
  sh[0][threadIdx.x] = s1; sh[1][threadIdx.x] = c1;
  sh[2][threadIdx.x] = s2; sh[3][threadIdx.x] = c2;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      double a1 = sh[0][threadIdx.x], b1 = sh[1][threadIdx.x];
      neumaier_merge(a1, b1, sh[0][threadIdx.x + off], sh[1][threadIdx.x + off]);
      double a2 = sh[2][threadIdx.x], b2 = sh[3][threadIdx.x];
      neumaier_merge(a2, b2, sh[2][threadIdx.x + off], sh[3][threadIdx.x + off]);
      sh[0][threadIdx.x] = a1; sh[1][threadIdx.x] = b1;
      sh[2][threadIdx.x] = a2; sh[3][threadIdx.x] = b2;
    }
    __syncthreads();
  }
  // counts are small integers: exact in double; reduce with a plain tree
  __shared__ double shc[256];
  shc[threadIdx.x] = cnt;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) shc[threadIdx.x] += shc[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sh[0][0] + sh[1][0];
    out[1] = sh[2][0] + sh[3][0];
    out[2] = shc[0];
  }
}

__global__ void __launch_bounds__(256) reduce_kernel(int n, const double* x, double* out) {
  reduce_body(n, x, out);
}

// Compensated FP64 sums of products of rows: block (a, b) sums x[a][w] *
// y[b][w] over w (y = null: x[a][w] alone) and counts the finite terms,
// out[2 (a B + b)] and out[2 (a B + b) + 1]; non-finite terms are skipped.
// The partial sums of the 256 threads meet in a fixed tree (deterministic).
__global__ void __launch_bounds__(256) pair_sums_kernel(int B, int W, const double* x, const double* y,
                                                        double* out) {
  __shared__ double sh[3][256];
  const int a = blockIdx.x / B, b = blockIdx.x % B;
  const double* xa = x + (size_t)a * W;
  const double* yb = y ? y + (size_t)b * W : nullptr;
  double s = 0, c = 0, cnt = 0;
  for (int i = threadIdx.x; i < W; i += 256) {
    const double v = yb ? xa[i] * yb[i] : xa[i];
    if (!isfinite(v)) continue;
    neumaier_add(s, c, v);
    cnt += 1.0;
  }
  sh[0][threadIdx.x] = s; sh[1][threadIdx.x] = c; sh[2][threadIdx.x] = cnt;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      double s1 = sh[0][threadIdx.x], c1 = sh[1][threadIdx.x];
      neumaier_merge(s1, c1, sh[0][threadIdx.x + off], sh[1][threadIdx.x + off]);
      sh[0][threadIdx.x] = s1; sh[1][threadIdx.x] = c1;
      sh[2][threadIdx.x] += sh[2][threadIdx.x + off];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * (size_t)blockIdx.x] = sh[0][0] + sh[1][0];
    out[2 * (size_t)blockIdx.x + 1] = sh[2][0];
  }
}

// ============================================================================
// batches, dual Monte Carlo
// ============================================================================
__global__ void __launch_bounds__(256) combine_persistent(const CombineArgs* descs, const int4* items,
                                                          int n_items, int* counter) {
  __shared__ int s_item;
  for (;;) {
    const int it = next_item(counter, &s_item);
    if (it >= n_items) break;
    const int4 w = items[it];
    const CombineArgs a = descs[w.x];
    combine_body(a, w.y);
    __syncthreads();
  }
}

// one block per RTT: out[3*b .. 3*b+2] = compensated sum, sum of squares, count
__global__ void __launch_bounds__(256) reduce_many(const int* n, const double* const* x, double* out) {
  reduce_body(n[blockIdx.x], x[blockIdx.x], out + 3 * blockIdx.x);
}

// Dual Monte Carlo estimators for one target state b, walkers sampled from
// P^a: ratio = psi^b / psi^a and the mixed local energy
// sum_t H_st psi^b(t) / psi^a(s) = ratio * E_loc^b(s), from both states'
// log|psi| and signs and b's local energy.  A walker whose sampled or target
// amplitude is zero or non-finite gets NaN and status -5; `first` starts the
// status, later targets fold into it.
__global__ void __launch_bounds__(256) mixed_kernel(int W, const double* la, const int8_t* sa,
                                                    const double* lb, const int8_t* sb, const double* eb,
                                                    const int32_t* stb, double* ratio, double* mixed,
                                                    int32_t* status, int first) {
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= W) return;
  const bool ok = stb[w] == 0 && sa[w] != 0 && sb[w] != 0 && isfinite(la[w]) && isfinite(lb[w]) &&
                  isfinite(eb[w]);
  const double r = ok ? (double)(sa[w] * sb[w]) * exp(lb[w] - la[w]) : NAN;
  ratio[w] = r;
  mixed[w] = ok ? r * eb[w] : NAN;
  if (status) {
    const int32_t st = ok ? 0 : -5;
    status[w] = first ? st : min(status[w], st);
  }
}

// graph-safe clearing of work counters (a kernel, not a memset node)
__global__ void fill_int(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void advance_u64(uint64_t* p, uint64_t by) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p += by;
}

}  // namespace rttk
