// Sequence-level mismatch statistics over a packed token stream (Section 4.2:
// the sequence-level rejection 1[S_seq <= tau_seq] with S_seq the sum of a
// Section 4.1 KL estimator (K1 or K3) of the correction ratio over a response,
// combined with the token-level truncation min(r_corr, tau_tok) as in the
// appendix's tis-srs-k1/k3-corr objectives).
//
// One workgroup per response: the token terms in fp64, summed in response_sum's
// order, which depends only on the response's length, so a response's score is
// bitwise the same wherever it sits in the stream. The token weights follow in
// a second pass over the tokens (the first left them in the cache): a rejected
// response then forms no exponentials for weights that become zero, and a call
// without weights none at all. Written in the first pass instead, 2000
// responses of 4000 tokens took 26 us rejected (16 here) and 18 us without
// weights (13).

#include "kernels.h"

namespace tim {
namespace {

template <int G>
__global__ __launch_bounds__(G * kChains) void seqstats_kernel(const float* __restrict__ a,
                                                               const float* __restrict__ b, int64_t T,
                                                               const int64_t* __restrict__ cu, int k3,
                                                               float C, double tau_seq, double* score,
                                                               uint8_t* keep, float* weight) {
  const int64_t j = blockIdx.x;
  // the response's tokens, clamped into [0, T]; reversed bounds give an empty response
  int64_t s0 = cu[j], s1 = cu[j + 1];
  s0 = s0 < 0 ? 0 : (s0 > T ? T : s0);
  s1 = s1 < s0 ? s0 : (s1 > T ? T : s1);
  const double S = response_sum<G>(s0, s1, [&](int64_t t) {
    const double delta = (double)a[t] - (double)b[t];  // exact in fp64
    return k3 ? k3_of_delta(delta) : -delta;           // K3 = (r - 1) - log r, K1 = -log r; r = e^delta
  });
  const bool k = S <= tau_seq;  // a NaN score rejects
  if (threadIdx.x == 0) {
    if (score) score[j] = S;
    if (keep) keep[j] = k ? 1 : 0;
  }
  if (!weight) return;
  constexpr int kStep = G * kChains;
  int64_t t = s0 + threadIdx.x;
  if (!k) {
    for (; t < s1; t += kStep) weight[t] = 0.f;
    return;
  }
  // kAhead tokens' loads issued together: 64 kept responses of 16384 tokens 26 us on one block of threads, 36 a token
  // at a time. `full`: all of them are the response's; else (the last, once) a load past its end takes the first one's.
  constexpr int kAhead = 4;
  auto weights = [&](bool full) {
    double delta[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int64_t u = full || t + i * kStep < s1 ? t + i * kStep : t;
      delta[i] = (double)a[u] - (double)b[u];
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (full || t + i * kStep < s1) weight[t + i * kStep] = tis_weight(delta[i], C);  // tim_mismatch's, truncated
  };
  for (; t + (kAhead - 1) * kStep < s1; t += kAhead * kStep) weights(true);
  if (t < s1) weights(false);
}

}  // namespace

hipError_t launch_mismatch_seq(const float* a, const float* b, int64_t T, const int64_t* cu_seqlens,
                               int64_t n_seq, bool k3, float C, double tau_seq, double* score,
                               uint8_t* keep, float* weight, hipStream_t s) {
  if (n_seq <= 0) return hipSuccess;
  if (n_seq > 0x7fffffff) return hipErrorInvalidValue;
  const bool four =
      response_blocks(k3 ? ResponseTerm::kK3 : ResponseTerm::kK1, T, n_seq, device_cu_count()) > 1;
  for (int64_t j = 0; j < n_seq; j += kLaunchResponses) {
    const dim3 g((unsigned)(n_seq - j < kLaunchResponses ? n_seq - j : kLaunchResponses));
    double* sc = score ? score + j : nullptr;
    uint8_t* kp = keep ? keep + j : nullptr;
    if (four)
      hipLaunchKernelGGL(seqstats_kernel<4>, g, dim3(4 * kChains), 0, s, a, b, T, cu_seqlens + j, k3 ? 1 : 0, C,
                         tau_seq, sc, kp, weight);
    else
      hipLaunchKernelGGL(seqstats_kernel<1>, g, dim3(kChains), 0, s, a, b, T, cu_seqlens + j, k3 ? 1 : 0, C, tau_seq,
                         sc, kp, weight);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tim
