// Confidence-based token fusion (Algorithm 1, TokenFusion; Eq. 4 first line of the paper):
// at every draft position keep the token whose own drafter gave it the highest
// probability.  The optional MIXTURE mode forms the confidence-weighted average of the
// drafters' distributions (the "weighted averaging" ensemble of Section 2.2).
#include "common.h"
#include "kernels.h"

#include <algorithm>

namespace specv {

// One position: the token with the highest confidence (the lowest drafter among equals).
__device__ __forceinline__ void fuse_position(int pos, bool used, int N, const float* __restrict__ conf, const int32_t* __restrict__ toks,
                                              int mixture, int32_t* __restrict__ fused, int32_t* __restrict__ winner,
                                              int32_t* __restrict__ q_row) {
  if (!used) {
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

__global__ void fuse_argmax_kernel(int B, int k_max, int N, const int32_t* __restrict__ k_len,
                                   const float* __restrict__ conf, const int32_t* __restrict__ toks,
                                   int mixture, int32_t* __restrict__ fused, int32_t* __restrict__ winner,
                                   int32_t* __restrict__ q_row) {
  const int pos = blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= B * k_max) return;
  const int b = pos / k_max, i = pos % k_max;
  fuse_position(pos, i < k_len[b], N, conf, toks, mixture, fused, winner, q_row);
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

// MIXTURE in one launch, every logit read once: a workgroup takes a segment of the vocabulary (2048 G classes) of one
// position, all its drafters' logits in registers.  It takes the segment's statistics of every drafter, posts them to
// the position's other workgroups as words {data : tag} (the call's own tag: nothing clears them), gathers theirs, and
// averages the exponentials that it still holds: a thread's are relative to its own maximum and take one fp64 factor per
// drafter.  A record that does not come within `patience` polls is worked out by the workgroup that misses it, from
// the logits and with the same arithmetic.
//
// What bounds it: memory (74 MB for 32 requests x 6 positions x 4 drafters x 32000 classes: 22 us with the gap to the next
// launch, three launches 29.5), then the vector unit, a dozen instructions per logit.  Four waves per workgroup: with
// eight the same registers hold 24.1 us' worth, because fewer workgroups are there to load while others wait.
constexpr int kOnceThreads = 256;
constexpr int kOnceWaves = kOnceThreads / kWave;
constexpr int kOnceBlock = kOnceThreads * 8;
constexpr int kOnceMaxN = 6;                     // drafters
constexpr int kOnceMaxRecords = 96;             // drafters x segments at most (once_fits): a thread gathers one

// Exponentials of n_rows (at most N) rows' logits in this thread's classes, relative to the thread's maximum m[n]; each wave's
// (maximum, sum) of every row go to LDS.
template <int DT, int N, int G>
__device__ __forceinline__ void once_exponentials(const void* __restrict__ logits, const Raw8<DT, G> (&raw)[N], int n_rows, int e_seg, int V,
                                                  float c, float (*sh_m)[kOnceWaves], double (*sh_z)[kOnceWaves], float (&e)[N][G][8],
                                                  float (&m)[N], int64_t row0) {
  const int tid = threadIdx.x, wave = tid >> 6;
#pragma unroll
  for (int n = 0; n < N; ++n) {
    m[n] = -INFINITY;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 8; ++j) e[n][g][j] = 0.f;
    if (n < n_rows) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        take8<false>(logits, (row0 + n) * V, e_seg + g * kOnceBlock + tid * 8, V, raw[n], g, e[n][g]);
#pragma unroll
        for (int j = 0; j < 8; ++j) m[n] = fmaxf(m[n], e[n][g][j]);
      }
      const float mm = (m[n] == -INFINITY) ? 0.f : m[n];
      float sum = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          e[n][g][j] = fast_exp2((e[n][g][j] - mm) * c);
          sum += e[n][g][j];
        }
      const float wm = wave_max(m[n]), wmm = (wm == -INFINITY) ? 0.f : wm;
      double z = static_cast<double>(sum) * static_cast<double>(fast_exp2((mm - wmm) * c));
      if (m[n] == -INFINITY) z = 0.0;
      sh_m[n][wave] = wm;                        // every lane stores the same value
      sh_z[n][wave] = wave_sum(z);
    }
    __builtin_amdgcn_sched_barrier(0);           // (rows side by side: twice the registers)
  }
}

// NB: drafters held (N of them exist); G: groups of eight classes per thread.
template <int DT, int NB, int G>
__global__ __launch_bounds__(kOnceThreads, NB <= 4 ? 4 : 3) void fuse_mixture_once_kernel(
    int k_max, int N, int V, int S, const int32_t* __restrict__ k_len, const float* __restrict__ conf,
    const int32_t* __restrict__ toks, const void* __restrict__ logits, float c, unsigned long long* __restrict__ msg, unsigned long long tag,
    int patience, int32_t* __restrict__ fused, int32_t* __restrict__ winner, int32_t* __restrict__ q_row, float* __restrict__ out) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef f4 f4_any __attribute__((aligned(4)));
  __shared__ float sh_m[NB][kOnceWaves];
  __shared__ double sh_z[NB][kOnceWaves];
  __shared__ float sh_rm[kOnceMaxRecords];
  __shared__ double sh_rz[kOnceMaxRecords];
  __shared__ unsigned char sh_have[kOnceMaxRecords];
  __shared__ float sh_row_m[NB];
  __shared__ double sh_row_w[NB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int seg = blockIdx.x % S, pos = blockIdx.x / S;
  const int b = pos / k_max;
  const bool used = pos - b * k_max < k_len[b];
  const int64_t row0 = static_cast<int64_t>(pos) * N;
  if (used) {
    const int e_seg = seg * G * kOnceBlock;
    Raw8<DT, G> raw[NB];
    auto e0 = [&](int sg) { return [=](int g) { return sg * G * kOnceBlock + g * kOnceBlock + tid * 8; }; };
#pragma unroll
    for (int n = 0; n < NB; ++n)       // (drafters past the last repeat it)
      issue8(logits, [&](int) { return (row0 + min(n, N - 1)) * V; }, e0(seg), V, raw[n]);
    double csum = 0.0;
    for (int n = 0; n < N; ++n) csum += static_cast<double>(conf[row0 + n]);
    float e[NB][G][8], m[NB];
    once_exponentials<DT, NB, G>(logits, raw, N, e_seg, V, c, sh_m, sh_z, e, m, row0);
    __syncthreads();
    // ---- records of this segment out (thread n: drafter n's), those of the others in (thread r: drafter r / S, segment r % S) ----
    const int n_rec = N * S;
    if (tid < N * kRecordWords) {                // (a thread per word of drafter n's)
      const int n = tid / kRecordWords, k = tid % kRecordWords;
      float M;
      double Z;
      merge_waves<kOnceWaves>(sh_m[n], sh_z[n], c, M, Z);
      const int r = n * S + seg;
      if (k == 0) { sh_rm[r] = M; sh_rz[r] = Z; sh_have[r] = 1; }
      if (S > 1) st_dev(msg + (row0 * S + r) * kRecordWords + k, message_word(k, Z, M, tag));
    }
    bool have = true;
    if (S > 1 && tid < (n_rec + kWave - 1) / kWave * kWave) {   // (wave-uniform)
      const bool want = tid < n_rec && tid % S != seg;
      const unsigned long long* from = msg + (row0 * S + tid) * kRecordWords;
      unsigned long long w[kRecordWords] = {0ull, 0ull, 0ull, 0ull};
      for (int poll = 0;; ++poll) {
        have = true;
        if (want) {
#pragma unroll
          for (int k = 0; k < record_words(DT); ++k) w[k] = ld_dev(from + k);
          have = have_tag<record_words(DT)>(w, tag);
        }
        if (__all(have) || poll >= patience) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (want) {
        sh_rm[tid] = message_max<record_words(DT)>(w);
        sh_rz[tid] = message_sum(w);
        sh_have[tid] = have;
      }
    }
    if (__syncthreads_or(!have)) {
      for (int r = 0; r < n_rec; ++r) {
        if (sh_have[r]) continue;
        const int n = r / S, sg = r - n * S;
        Raw8<DT, G> one[1];
        issue8(logits, [&](int) { return (row0 + n) * V; }, e0(sg), V, one[0]);
        float e1[1][G][8], m1[1];
        once_exponentials<DT, 1, G>(logits, one, 1, sg * G * kOnceBlock, V, c, sh_m, sh_z, e1, m1, row0 + n);
        __syncthreads();
        if (tid == 0) merge_waves<kOnceWaves>(sh_m[0], sh_z[0], c, sh_rm[r], sh_rz[r]);
        __syncthreads();
      }
    }
    // ---- every drafter's maximum and weight / sum: groups of 16 lanes ----
    if (wave * 4 < N) {
      const int n = tid >> 4, sl = tid & 15;
      float rm;
      double rz;
      merged_stats([&](int sg) -> SegStat {
        SegStat st;
        st.m = sh_rm[n * S + sg]; st.pad = 0.f; st.z = sh_rz[n * S + sg];
        return st;
      }, n < N ? S : 0, c, sl, rm, rz);
      if (sl == 0 && n < N) {
        const double w = (csum > 0.0) ? static_cast<double>(conf[row0 + n]) / csum : 1.0 / N;
        sh_row_m[n] = rm;
        sh_row_w[n] = w / rz;
      }
    }
    __syncthreads();
    double acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[g][j] = 0.0;
#pragma unroll
    for (int n = 0; n < NB; ++n)
      if (n < N) {
        // (a thread without a finite logit of this drafter has exponentials 0 and takes the row's maximum for its own: a factor
        // from any fixed number overflows where the row lies far below it, and 0 x inf is no probability)
        const float row_m = sh_row_m[n];
        const double f = sh_row_w[n] * exp2(static_cast<double>((m[n] == -INFINITY ? row_m : m[n]) - row_m) * static_cast<double>(c));
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            asm volatile("" : "+v"(e[n][g][j]));       // (else converted to fp64 where it is made, and held so)
            acc[g][j] += f * static_cast<double>(e[n][g][j]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int at0 = e_seg + g * kOnceBlock + tid * 8;
      if (at0 < V) {
        const int at = first8(at0, V);        // class of acc[g][0]
        float* o = out + static_cast<int64_t>(pos) * V + at;
        if (at == at0 && V >= 8) {
          f4 x, y;
#pragma unroll
          for (int j = 0; j < 4; ++j) { x[j] = static_cast<float>(acc[g][j]); y[j] = static_cast<float>(acc[g][4 + j]); }
          *reinterpret_cast<f4_any*>(o) = x;
          *reinterpret_cast<f4_any*>(o + 4) = y;
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) if (at + j >= at0 && at + j < V) o[j] = static_cast<float>(acc[g][j]);
        }
      }
    }
  }
  if (seg == 0 && tid == 0) fuse_position(pos, used, N, conf, toks, 1, fused, winner, q_row);
}

// Classes per workgroup and records of the one-launch kernel.
constexpr int kOnceGroups = 2;
static int once_segments(int N, int V) { return (V + kOnceGroups * kOnceBlock - 1) / (kOnceGroups * kOnceBlock); }
static size_t once_bytes(int B, int k_max, int N, int V) {
  return static_cast<size_t>(B) * k_max * N * once_segments(N, V) * kRecordWords * sizeof(unsigned long long);
}
// Kernel plus gaps, one launch / statistics, average and fusion (us): 32 x 6 positions x 4 drafters x 32000 classes 22.4 / 29.5
// (74 MB), 2 drafters 16.0 / 21.5, 6 drafters 30.1 / 35.8, fp32 28.5 / 42.1, 32 x 16 x 4 x 32000 49.7 / 66.7, 16 x 6 x 4 x 65536
// 24.7 / 29.1, 16 x 6 x 6 x 65536 33.6 / 36.0, 16 x 6 x 2 x 128256 30.8 / 32.9.  Many workgroups that wait for each other over many
// records lose: 16 x 6 x 3 x 128256 50.2 / 40.9, x 4 60.4 / 49.2; so do more drafters than leave two workgroups a place on
// a compute unit (8 x 32000: 46.0 / 43.4).
static bool once_fits(int N, int V) {
  const int S = once_segments(N, V);
  return N <= kOnceMaxN && (S <= 16 || N * S <= 64);
}

template <int DT>
static auto once_kernel(int N) {
  return N <= 2 ? fuse_mixture_once_kernel<DT, 2, 2> : (N <= 4 ? fuse_mixture_once_kernel<DT, 4, 2>
       : fuse_mixture_once_kernel<DT, 6, 2>);
}

size_t fuse_workspace_min_bytes(int B, int k_max, int N, int V, int mode) {
  if (mode != 1) return 0;
  return static_cast<size_t>(B) * k_max * N * stats_segments(V) * sizeof(SegStat) + 256;
}

size_t fuse_workspace_bytes(int B, int k_max, int N, int V, int mode) {
  const size_t least = fuse_workspace_min_bytes(B, k_max, N, V, mode);
  return mode == 1 && once_fits(N, V) ? std::max(least, once_bytes(B, k_max, N, V)) : least;
}

void launch_fuse(const FuseArgs& a, hipStream_t stream) {
  const int positions = a.B * a.k_max;
  if (positions <= 0) return;
  const float c = kLog2e / a.temperature;
  // One launch wherever a workgroup holds the logits of all drafters and the workspace (the size query's, not the least that
  // is taken) has room for the records.
  if (a.mode == 1 && once_fits(a.N, a.V) && static_cast<int64_t>(positions) * once_segments(a.N, a.V) <= INT32_MAX / kOnceThreads && a.workspace_bytes >= once_bytes(a.B, a.k_max, a.N, a.V)) {
    const int S = once_segments(a.N, a.V);
    unsigned long long* msg = static_cast<unsigned long long*>(a.workspace);
    const MessageTag t = S > 1 ? next_message_tag(false, stream) : MessageTag{};
    if (t.clear)
      clear_messages(msg, static_cast<int64_t>(once_bytes(a.B, a.k_max, a.N, a.V) / sizeof(unsigned long long)), stream);
    hipLaunchKernelGGL((a.l_dtype == kBF16 ? once_kernel<kBF16>(a.N) : once_kernel<kF32>(a.N)), dim3(static_cast<unsigned>(positions) * S),
                       dim3(kOnceThreads), 0, stream, a.k_max, a.N, a.V, S, a.k_len, a.conf, a.draft_tokens, a.draft_logits, c, msg,
                       t.tag,
                       a.patience >= 0 && a.patience <= 1000000 ? a.patience : 1000, a.fused_token, a.winner, a.q_row, a.fused_probs);
    return;
  }
  hipLaunchKernelGGL(fuse_argmax_kernel, dim3((positions + 255) / 256), dim3(256), 0, stream, a.B, a.k_max,
                     a.N, a.k_len, a.conf, a.draft_tokens, a.mode == 1, a.fused_token, a.winner, a.q_row);
  if (a.mode != 1) return;
  SegStat* stats = static_cast<SegStat*>(a.workspace);
  // statistics of every drafter row (rows of unused positions are computed but never read)
  launch_row_stats(a.draft_logits, a.l_dtype, positions * a.N, nullptr, kBF16, 0, a.V, c, stats, stream);
  const int nseg = stats_segments(a.V);
  dim3 grid((a.V + kMixSeg - 1) / kMixSeg, positions);
  hipLaunchKernelGGL((a.l_dtype == kBF16 ? fuse_mixture_kernel<kBF16> : fuse_mixture_kernel<kF32>), grid, dim3(kMixThreads), 0, stream,
                     a.k_max, a.N, a.V, a.k_len, a.conf, a.draft_logits, c, nseg, stats, a.fused_probs);
}

}  // namespace specv
