// Drop-set stability signals of the routing decisions (paper section 3.4, UCS
// operators (3) diffusion-head cache reuse and (4) denoising-step early exit).
//
// For each sequence, the drop set D_t of a timestep is its routable tokens
// (not always-kept) with token_pos < 0. Between two timesteps:
//   J    = |D_t n D_ref| / |D_t u D_ref|          (Eq. 10; 1 for an empty union)
//   J_rd = E[J] for two independent uniformly random subsets of the routable
//          tokens with the same sizes (hypergeometric overlap)
//   RDA  = (J - J_rd) / (1 - J_rd)                 (Eq. 11; 1 when J_rd = 1)
//
// One workgroup per sequence: the four counts (routable, dropped at t, dropped
// at t_ref, dropped at both) are reduced over the block, J is formed from the
// integers and J_rd in fp64 by the whole block. The overlap X of the two random
// sets is hypergeometric with mean E = a b / n; by Hoeffding's inequality for
// sampling without replacement, P(|X - E| >= s) <= 2 exp(-2 s^2 / m) with
// m = min(a, b), so the window E +- sqrt(48 m) misses less than 1e-41 of the
// mass. Four threads take a contiguous run of that window: the probability at
// the run's point nearest the mode comes from lgamma, the others from the
// exact ratio of consecutive terms walking away from it, one thread each way
// (so the terms only shrink and an underflow to zero is harmless). The
// per-thread sums are then added in a fixed order. Bound: latency, a few loads
// in flight together and one lgamma.
#include "ce_device.hpp"
#include "ce_host.hpp"
#include "ce_launch.hpp"
#include "ce_router.h"

namespace ce {

namespace {

__device__ double jaccard_of(int64_t x, int64_t a, int64_t b) {
  const int64_t u = a + b - x;
  return u == 0 ? 1.0 : (double)x / (double)u;
}

// E[J] over the window (see above); every thread calls it, thread 0 gets the
// sum. ln P(x) = ln C(a, x) + ln C(n - a, b - x) - ln C(n, b) takes nine
// lgammas, five of them the same for every x: the four threads of a run take
// one of its four each and eight spare threads the five, so the chain is one
// lgamma long and not nine.
template <int kThreads>
__device__ double expected_random_jaccard(int64_t n, int64_t a, int64_t b, int tid, double* common, double* part) {
  constexpr int kRuns = kThreads / 4 - 2;  // runs of the window: four threads each, two quads left
  int64_t xlo = a + b - n > 0 ? a + b - n : 0;
  int64_t xhi = a < b ? a : b;
  const double mean = (double)a * (double)b / (double)(n > 0 ? n : 1);
  const double half = sqrt(48.0 * (double)xhi) + 2.0;
  const int64_t wlo = (int64_t)floor(mean - half), whi = (int64_t)ceil(mean + half);
  xlo = wlo > xlo ? wlo : xlo;
  xhi = whi < xhi ? whi : xhi;
  const int run = tid >> 2, q4 = tid & 3;
  const int64_t per = (xhi - xlo + kRuns) / kRuns;
  const int64_t c0 = xlo + (int64_t)run * per;
  const int64_t c1 = c0 + per - 1 < xhi ? c0 + per - 1 : xhi;
  const bool mine = run < kRuns && c0 <= c1;
  const int64_t xm = (int64_t)(((double)(a + 1) * (double)(b + 1)) / (double)(n + 2));
  const int64_t x0 = xm < c0 ? c0 : (xm > c1 ? c1 : xm);
  const int spare = tid - 4 * kRuns;
  double arg = 1.0;
  if (mine) arg = (double)(q4 == 0 ? x0 : q4 == 1 ? a - x0 : q4 == 2 ? b - x0 : n - a - b + x0) + 1.0;
  else if (spare >= 0)
    arg = (double)(spare == 0 ? a : spare == 1 ? n - a : spare == 2 ? n : spare == 3 ? b : n - b) + 1.0;
  const double lg = lgamma(arg);
  if (spare >= 0 && spare < 5) common[spare] = lg;
  const int lane = threadIdx.x & 63, l0 = lane & ~3;
  const double lx = __shfl(lg, l0), lax = __shfl(lg, l0 + 1), lbx = __shfl(lg, l0 + 2), lr = __shfl(lg, l0 + 3);
  __syncthreads();
  double sum = 0.0;
  if (mine && q4 < 2) {
    const double p0 = exp((common[0] - lx - lax) + (common[1] - lbx - lr) - (common[2] - common[3] - common[4]));
    const double c = (double)(n - a - b);
    double q = p0;
    if (p0 == 0.0) {
    } else if (q4 == 0) {
      sum = p0 * jaccard_of(x0, a, b);
      for (int64_t x = x0; x < c1; ++x) {  // P(x + 1) / P(x) = (a - x)(b - x) / ((x + 1)(n - a - b + x + 1))
        q *= ((double)(a - x) * (double)(b - x)) / ((double)(x + 1) * (c + (double)(x + 1)));
        sum += q * jaccard_of(x + 1, a, b);
      }
    } else {
      for (int64_t x = x0; x > c0; --x) {  // P(x - 1) / P(x) = x (n - a - b + x) / ((a - x + 1)(b - x + 1))
        q *= ((double)x * (c + (double)x)) / ((double)(a - x + 1) * (double)(b - x + 1));
        sum += q * jaccard_of(x - 1, a, b);
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == 0) part[tid >> 6] = sum;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kThreads / 64; ++w) t += part[w];
  return t;
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void stability_kernel(const int32_t* __restrict__ offs,
                                                        const uint8_t* __restrict__ flags, int T,
                                                        const int32_t* __restrict__ tp_t,
                                                        const int32_t* __restrict__ tp_r,
                                                        float* __restrict__ jac,
                                                        float* __restrict__ jrand,
                                                        float* __restrict__ rda) {
  constexpr int kWaves = kThreads / 64;
  __shared__ int cnt[kWaves][4];
  __shared__ double part[kWaves];
  __shared__ double common[5];
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  int o0 = offs[b], o1 = offs[b + 1];
  const int lo = o0 < 0 ? 0 : (o0 > T ? T : o0);
  const int hi = o1 < lo ? lo : (o1 > T ? T : o1);
  int n = 0, na = 0, nb = 0, nx = 0;
  // four tokens per thread and step, their loads in flight together
  for (int i0 = lo + tid; i0 < hi; i0 += 4 * kThreads) {
    uint8_t f[4];
    int32_t pt[4], pr[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = min(i0 + k * kThreads, hi - 1);
      f[k] = flags[i];
      pt[k] = tp_t[i];
      pr[k] = tp_r[i];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = i0 + k * kThreads < hi && !(f[k] & CE_TOK_KEEP);
      n += in;
      na += in && pt[k] < 0;
      nb += in && pr[k] < 0;
      nx += in && pt[k] < 0 && pr[k] < 0;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    n += __shfl_xor(n, o);
    na += __shfl_xor(na, o);
    nb += __shfl_xor(nb, o);
    nx += __shfl_xor(nx, o);
  }
  if ((tid & 63) == 0) {
    cnt[tid >> 6][0] = n;
    cnt[tid >> 6][1] = na;
    cnt[tid >> 6][2] = nb;
    cnt[tid >> 6][3] = nx;
  }
  __syncthreads();
  int64_t c[4];
  for (int k = 0; k < 4; ++k) {
    c[k] = 0;
    for (int w = 0; w < kWaves; ++w) c[k] += cnt[w][k];
  }
  // c[0] = routable tokens, c[1] / c[2] = dropped at t / t_ref, c[3] = dropped at both
  double jr;
  const int64_t xlo = c[1] + c[2] - c[0] > 0 ? c[1] + c[2] - c[0] : 0;
  const int64_t xhi = c[1] < c[2] ? c[1] : c[2];
  if (xlo >= xhi) {
    jr = jaccard_of(xlo, c[1], c[2]);  // a single possible overlap
  } else {
    jr = expected_random_jaccard<kThreads>(c[0], c[1], c[2], tid, common, part);
  }
  if (tid != 0) return;
  const double j = jaccard_of(c[3], c[1], c[2]);
  jac[b] = (float)j;
  if (jrand) jrand[b] = (float)jr;
  if (rda) rda[b] = (float)(jr >= 1.0 ? 1.0 : (j - jr) / (1.0 - jr));
}

}  // namespace

hipError_t launch_stability(const int32_t* seq_offsets, const uint8_t* flags, int B, int T,
                            const int32_t* tp_t, const int32_t* tp_ref, float* jaccard, float* j_rand,
                            float* rda, hipStream_t stream) {
  if (B <= 0) return hipSuccess;
  // 1024 threads each only for long sequences: the lgammas of a wider workgroup
  // cost more than its shorter loops save. Stability and the layer gap at d 1536
  // in turn, us, with 256 and 1024 threads: 1 x 300 tokens 11.7 and 13.4, 4 x 1000
  // 14.9 and 16.7, 4 x 2000 22.9 and 23.6, three of 1341, 3379 and 1224 21.3 and
  // 20.9, 16 x 3000 59.5 and 58.7, 4 x 4224 32.9 and 31.8; two workgroups to a CU,
  // 512 x 500 alone: 7.9 and 16 (256 threads with one token a step and nine
  // lgammas each: 12)
  constexpr int kWide = 1792;
  if (wide_signal(B, T, kWide))
    hipLaunchKernelGGL(stability_kernel<1024>, dim3(B), dim3(1024), 0, stream, seq_offsets, flags, T, tp_t, tp_ref,
                       jaccard, j_rand, rda);
  else
    hipLaunchKernelGGL(stability_kernel<256>, dim3(B), dim3(256), 0, stream, seq_offsets, flags, T, tp_t, tp_ref,
                       jaccard, j_rand, rda);
  return hipGetLastError();
}

}  // namespace ce
