// Confidence-based token fusion (Algorithm 1, TokenFusion; Eq. 4 first line of the paper):
// at every draft position keep the token whose own drafter gave it the highest
// probability.  The optional MIXTURE mode forms the confidence-weighted average of the
// drafters' distributions (the "weighted averaging" ensemble of Section 2.2).
#include "common.h"
#include "kernels.h"

namespace specv {

__global__ void fuse_argmax_kernel(int B, int k_max, int N, const int32_t* __restrict__ k_len,
                                   const float* __restrict__ conf, const int32_t* __restrict__ toks,
                                   int mixture, int32_t* __restrict__ fused, int32_t* __restrict__ winner,
                                   int32_t* __restrict__ q_row) {
  const int pos = blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= B * k_max) return;
  const int b = pos / k_max, i = pos % k_max;
  if (i >= k_len[b]) {
    fused[pos] = -1; winner[pos] = -1; q_row[pos] = -1;
    return;
  }
  const float* c = conf + static_cast<int64_t>(pos) * N;
  int best = 0;
  float bv = c[0];
  for (int n = 1; n < N; ++n) {
    const float v = c[n];
    if (v > bv) { bv = v; best = n; }
  }
  winner[pos] = best;
  fused[pos] = toks[static_cast<int64_t>(pos) * N + best];
  q_row[pos] = mixture ? pos : pos * N + best;
}

// MIXTURE: fused_probs[pos, v] = sum_n w_n 2^((l_nv - m_n) c) / Z_n
// A workgroup takes 2048 classes of one position.  Groups of 16 lanes merge the statistics of one drafter row each and
// hand (max, w / Z) to the workgroup through LDS; meanwhile the logits of the first four drafters are on their way.
// Bound by memory: N logit rows in, one fp32 row out.  (Every thread merged the statistics of all drafters by itself
// before, two dozen fp64 exponentials per thread: 32 requests x 6 positions x 4 drafters x 32000 classes, 74 MB,
// 30.4 us; 17.4 us = 4.2 TB/s now.)
constexpr int kMixThreads = 256;
constexpr int kMixSeg = kMixThreads * 8;
constexpr int kMixRound = kMixThreads / 16;      // drafters whose statistics are merged at once
constexpr int kMixFly = 4;                       // drafters whose logits are loaded together

template <int DT>
__global__ __launch_bounds__(kMixThreads) void fuse_mixture_kernel(
    int k_max, int N, int V, const int32_t* __restrict__ k_len, const float* __restrict__ conf,
    const void* __restrict__ logits, float c, int nseg, const SegStat* __restrict__ stats,
    float* __restrict__ out) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef f4 f4_any __attribute__((aligned(4)));
  __shared__ float sh_m[kMixRound];
  __shared__ double sh_w[kMixRound];
  const int pos = blockIdx.y, tid = threadIdx.x;
  const int b = pos / k_max, i = pos % k_max;
  const int e0 = (blockIdx.x * kMixThreads + tid) * 8;
  const int64_t row0 = static_cast<int64_t>(pos) * N;
  if (i >= k_len[b]) return;
  double acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.0;
  Raw8<DT, kMixFly> raw;
  int n_at = 0;                       // first drafter of the group on its way
  auto off = [&](int u) { return (row0 + min(n_at + u, N - 1)) * V; };      // (drafters past the last repeat it)
  auto load = [&](int n0) {
    n_at = n0;
    issue8(logits, off, [&](int) { return e0; }, V, raw);
  };
  load(0);
  for (int r0 = 0; r0 < N; r0 += kMixRound) {
    const int g = r0 + (tid >> 4), sl = tid & 15;
    const bool mine = g < N;
    float M;
    double Z;
    merged_row_stats<false>(stats + (row0 + (mine ? g : 0)) * nseg, mine ? nseg : 0, c, sl, M, Z);
    __syncthreads();                  // earlier readers of sh_m and sh_w are done
    if (sl == 0 && mine) {
      double csum = 0.0;
      for (int n = 0; n < N; ++n) csum += static_cast<double>(conf[row0 + n]);
      const double w = (csum > 0.0) ? static_cast<double>(conf[row0 + g]) / csum : 1.0 / N;
      sh_m[tid >> 4] = M;
      sh_w[tid >> 4] = w / Z;
    }
    __syncthreads();
    for (int n0 = r0; n0 < min(N, r0 + kMixRound); n0 += kMixFly) {
      if (n0 > 0) load(n0);
#pragma unroll
      for (int u = 0; u < kMixFly; ++u)
        if (n0 + u < N) {
          const float m = sh_m[n0 + u - r0];
          const double wz = sh_w[n0 + u - r0];
          float x[8];
          take8<true>(logits, off(u), e0, V, raw, u, x);
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[j] += wz * static_cast<double>(fast_exp2((x[j] - m) * c));
        }
    }
  }
  if (e0 >= V) return;
  const int at = first8(e0, V);        // class of acc[0]
  float* o = out + static_cast<int64_t>(pos) * V + at;
  if (at == e0 && V >= 8) {
    f4 a, d;
#pragma unroll
    for (int j = 0; j < 4; ++j) { a[j] = static_cast<float>(acc[j]); d[j] = static_cast<float>(acc[4 + j]); }
    *reinterpret_cast<f4_any*>(o) = a;
    *reinterpret_cast<f4_any*>(o + 4) = d;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) if (at + j >= e0 && at + j < V) o[j] = static_cast<float>(acc[j]);
  }
}

size_t fuse_workspace_bytes(int B, int k_max, int N, int V, int mode) {
  if (mode != 1) return 0;
  return static_cast<size_t>(B) * k_max * N * stats_segments(V) * sizeof(SegStat) + 256;
}

void launch_fuse(const FuseArgs& a, hipStream_t stream) {
  const int positions = a.B * a.k_max;
  if (positions <= 0) return;
  hipLaunchKernelGGL(fuse_argmax_kernel, dim3((positions + 255) / 256), dim3(256), 0, stream, a.B, a.k_max,
                     a.N, a.k_len, a.conf, a.draft_tokens, a.mode == 1, a.fused_token, a.winner, a.q_row);
  if (a.mode != 1) return;
  const float c = kLog2e / a.temperature;
  SegStat* stats = static_cast<SegStat*>(a.workspace);
  // statistics of every drafter row (rows of unused positions are computed but never read)
  launch_row_stats(a.draft_logits, a.l_dtype, positions * a.N, nullptr, kBF16, 0, a.V, c, stats, stream);
  const int nseg = stats_segments(a.V);
  dim3 grid((a.V + kMixSeg - 1) / kMixSeg, positions);
  hipLaunchKernelGGL((a.l_dtype == kBF16 ? fuse_mixture_kernel<kBF16> : fuse_mixture_kernel<kF32>), grid, dim3(kMixThreads), 0, stream,
                     a.k_max, a.N, a.V, a.k_len, a.conf, a.draft_logits, c, nseg, stats, a.fused_probs);
}

}  // namespace specv
