// Vocab-wide softmax statistics and the acceptance-rejection walk (Section 2.1 of the
// paper: accept x_i when q_i(x_i) <= o_i(x_i), else reject with probability
// 1 - o_i(x_i)/q_i(x_i); replacement from norm(max(0, o_i - q_i)); bonus token when
// nothing is rejected), extended to sibling drafts of a tree by recursive rejection.
//
// Kernels:
//   row_stats_kernel      one workgroup per (row, vocab segment): segment maximum and
//                         sum of 2^((l-m)c).  Pure streaming, HBM-bound (64 x 128256 bf16 linear drafts 36.4 -> 30.6 us
//                         with the four loads of a thread in flight together; 5 x 50257 fp32 13.2 -> 4.1 us).
//   accept_walk_kernel    one master workgroup per request: the sequential walk; every full
//                         pass over a row pair (residual mass, inverse-CDF search) is
//                         spread over the workgroup's 16 waves and, for large vocabularies,
//                         over the waves of up to three helper workgroups.
//   accept_linear_kernel  linear drafts: the scalar tests repeated in every workgroup, the one
//                         vocabulary-wide draw spread over several workgroups per request.
//   row_stats_prog_kernel large batches of linear drafts: the statistics pass in chain order, with
//                         the accept decisions taken on the way, so that rows behind a request's
//                         first rejection are not read.
// (accept_cluster.hip holds the tree kernel that reads only the rows a walk reaches.)
// Up to 128 draft nodes per request; the children of one node share one draft row, the one the
// first child names.
#include "common.h"
#include "kernels.h"

#include <algorithm>
#include <chrono>

namespace specv {

// ----------------------------------------------------------------------------------
// messages between the workgroups of one launch
// ----------------------------------------------------------------------------------
static bool stream_captures(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

// Tags with rounds are below 2^36, those without have that bit set.
// The count starts somewhere else in every process: what memory held before it was the process's own is no message.
MessageTag next_message_tag(bool rounds, hipStream_t stream) {
  static const uint64_t start = static_cast<uint64_t>(std::chrono::steady_clock::now().time_since_epoch().count()) * 0x9E3779B97F4A7C15ull >> 20;
  static std::atomic<uint64_t> calls[2];
  const uint64_t n = calls[rounds].fetch_add(1, std::memory_order_relaxed);
  constexpr uint64_t kBit = 1ull << (kTagBits - 1), kRoundCalls = kBit / kTagRounds, kCalls = kBit;
  MessageTag t;
  const uint64_t at = (start + n) % (rounds ? kRoundCalls : kCalls);
  t.tag = rounds ? at * kTagRounds : kBit + at;
  t.clear = n >= (rounds ? kRoundCalls : kCalls) || stream_captures(stream);
  return t;
}

__global__ __launch_bounds__(256) void clear_messages_kernel(unsigned long long* __restrict__ words, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256) words[i] = 0ull;
}

void clear_messages(unsigned long long* words, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(clear_messages_kernel, dim3(static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, 512))), dim3(256), 0, stream, words, n);
}

// ----------------------------------------------------------------------------------
// row statistics
// ----------------------------------------------------------------------------------
constexpr int kStatThreads = 256;
constexpr int kStatPerThread = 32;                              // 4 x 8 elements
constexpr int kStatSeg = kStatThreads * kStatPerThread;         // 8192 logits per workgroup

int stats_segments(int V) { return (V + kStatSeg - 1) / kStatSeg; }

// (max, sum 2^((l - max) c)) of one 8192-logit segment of a row, by a workgroup of kStatThreads; the result is
// valid in thread 0, for which the function returns true.
struct StatScratch {
  float m[kStatThreads / kWave];
  double z[kStatThreads / kWave];
};
template <int DT>
__device__ __forceinline__ bool segment_stats(const void* __restrict__ base, int64_t row_off, int e_seg, int V, float c,
                                              StatScratch& sh, float& M_out, double& Z_out) {
  constexpr int kGroups = kStatPerThread / 8;
  float x[kGroups][8];
  {
    auto off = [&](int) { return row_off; };
    auto e0 = [&](int j) { return e_seg + (j * kStatThreads + static_cast<int>(threadIdx.x)) * 8; };
    Raw8<DT, kGroups> raw;
    issue8(base, off, e0, V, raw);
#pragma unroll
    for (int j = 0; j < kGroups; ++j) take8<false>(base, row_off, e0(j), V, raw, j, x[j]);
  }
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < kGroups; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, x[j][i]);
  const float mm = (m == -INFINITY) ? 0.f : m;
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < kGroups; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) s += fast_exp2((x[j][i] - mm) * c);

  // workgroup combine: maximum first, then rescaled sums in fp64
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float wm = wave_max(m);
  if (lane == 0) sh.m[wave] = wm;
  __syncthreads();
  float M = sh.m[0];
#pragma unroll
  for (int w = 1; w < kStatThreads / kWave; ++w) M = fmaxf(M, sh.m[w]);
  const float MM = (M == -INFINITY) ? 0.f : M;
  double z = static_cast<double>(s) * static_cast<double>(fast_exp2((mm - MM) * c));
  if (m == -INFINITY) z = 0.0;
  z = wave_sum(z);
  if (lane == 0) sh.z[wave] = z;
  __syncthreads();
  double Z = 0.0;
#pragma unroll
  for (int w = 0; w < kStatThreads / kWave; ++w) Z += sh.z[w];
  M_out = M;
  Z_out = Z;
  return threadIdx.x == 0;
}

__device__ __forceinline__ bool segment_stats(const void* __restrict__ base, int dtype, int64_t row_off, int e_seg, int V,
                                              float c, StatScratch& sh, float& M_out, double& Z_out) {
  return dtype == kBF16 ? segment_stats<kBF16>(base, row_off, e_seg, V, c, sh, M_out, Z_out)
                        : segment_stats<kF32>(base, row_off, e_seg, V, c, sh, M_out, Z_out);
}

__global__ __launch_bounds__(kStatThreads) void row_stats_kernel(
    const void* __restrict__ t_base, int t_dtype, int n_t_rows,
    const void* __restrict__ q_base, int q_dtype, int n_q_rows,
    int V, float c, int nseg, SegStat* __restrict__ stats, unsigned* __restrict__ zero_words, int n_zero,
    const int32_t* __restrict__ q_row) {
  const int seg = blockIdx.x;
  const int row = blockIdx.y;
  // side job of the first workgroup: clear the flags the walk kernel's workgroups exchange
  if (seg == 0 && row == 0)
    for (int i = threadIdx.x; i < n_zero; i += kStatThreads) zero_words[i] = 0u;
  const void* base = t_base;
  int dtype = t_dtype;
  int64_t r = row;
  if (row >= n_t_rows) {
    base = q_base; dtype = q_dtype; r = row - n_t_rows;
    // With more draft rows than draft nodes (several drafters per position) most rows are nobody's: the grid then has a row
    // per node, the one it was drawn from (clamped as the walk clamps it; nodes that share one write the same record).
    // 32 requests x 6 nodes, 4 drafters, 32000 classes: 10.8 us when every draft row had workgroups that looked
    // for a node of theirs first.
    if (q_row) r = min(max(q_row[r], 0), n_q_rows - 1);
  }
  const int64_t row_off = r * static_cast<int64_t>(V);
  __shared__ StatScratch sh;
  float M;
  double Z;
  if (segment_stats(base, dtype, row_off, seg * kStatSeg, V, c, sh, M, Z)) {
    SegStat st;
    st.m = M; st.pad = 0.f; st.z = Z;
    stats[(row < n_t_rows ? row : n_t_rows + r) * nseg + seg] = st;
  }
}

__global__ __launch_bounds__(kStatThreads) void zero_words_kernel(unsigned* __restrict__ words, int n) {
  for (int i = threadIdx.x; i < n; i += kStatThreads) words[i] = 0u;
}

void launch_row_stats(const void* t_base, int t_dtype, int n_t_rows, const void* q_base, int q_dtype,
                      int n_q_rows, int V, float c, SegStat* stats, hipStream_t stream, unsigned* zero_words,
                      int n_zero, const int32_t* q_row, int n_nodes) {
  const int rows = n_t_rows + (q_row ? n_nodes : n_q_rows);
  if (rows <= 0 || V <= 0) return;
  const int nseg = stats_segments(V);
  dim3 grid(nseg, rows);
  hipLaunchKernelGGL(row_stats_kernel, grid, dim3(kStatThreads), 0, stream, t_base, t_dtype,
                     n_t_rows, q_base, q_dtype, n_q_rows, V, c, nseg, stats, zero_words, n_zero, q_row);
}

// ----------------------------------------------------------------------------------
// walk
// ----------------------------------------------------------------------------------
constexpr int kWalkThreads = 1024;
constexpr int kWalkWaves = kWalkThreads / kWave;
constexpr int kMaxNodes = 128;
constexpr int kMaxBlocksPerSeg = 256;      // vocabularies up to 16 * 256 * 512 = 2M tokens

struct WalkRows {
  const void* t_base; int t_dtype; int64_t t_off; float t_m; double t_invz;   // target row
  const void* q_base; int q_dtype; int64_t q_off; float q_m; double q_invz;   // draft row
  int q_is_probs;
  int have_q;       // level 0 needs no draft row
};

// Weight of token class v at residual level L (L rejections so far at this node):
//   r_0 = p;  w_k = max(0, r_{k-1} - q);  r_k = w_k / R_k,  R_k = sum_v w_k(v).
// The weight of level L is w_L (unnormalised; p itself at level 0).  Per-class values are
// fp32 (their relative error, ~1e-7, is that of the hardware exp2 anyway); every sum over
// classes is carried in fp64.
// Weights of eight consecutive token classes from their logits (q: logits or probabilities).
// The level loop is outermost so that its (wave-uniform) trip count is tested once per eight classes;
// the last level stays unnormalised (scale 1, exact).
__device__ __forceinline__ void weights_from(const WalkRows& R, const float (&lp)[8], const float (&lq)[8],
                                             int n_valid, float c, int L, const float* __restrict__ inv_R,
                                             float (&w)[8]) {
  const float t_invz = static_cast<float>(R.t_invz), q_invz = static_cast<float>(R.q_invz);
  float q[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    w[j] = fast_exp2((lp[j] - R.t_m) * c) * t_invz;
    q[j] = 0.f;
    if (L > 0) q[j] = R.q_is_probs ? lq[j] : fast_exp2((lq[j] - R.q_m) * c) * q_invz;
  }
  for (int k = 0; k < L; ++k) {
    const float scale = (k + 1 < L) ? inv_R[k] : 1.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = fmaxf(w[j] - q[j], 0.f) * scale;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = (j < n_valid) ? w[j] : 0.f;
}

__device__ __forceinline__ void weights8(const WalkRows& R, int e0, int V, float c, int L,
                                         const float* __restrict__ inv_R, float (&w)[8]) {
  float lp[8], lq[8];
  load8(R.t_base, R.t_dtype, R.t_off, e0, V, lp);
  if (L > 0) load8(R.q_base, R.q_dtype, R.q_off, e0, V, lq);
  weights_from(R, lp, lq, min(8, V - e0), c, L, inv_R, w);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void unpack_bf16x8(u32x4 r, float (&x)[8]) {
  x[0] = bf16_lo(r[0]); x[1] = bf16_hi(r[0]); x[2] = bf16_lo(r[1]); x[3] = bf16_hi(r[1]);
  x[4] = bf16_lo(r[2]); x[5] = bf16_hi(r[2]); x[6] = bf16_lo(r[3]); x[7] = bf16_hi(r[3]);
}

// Sum of the level-L weights over [e_begin, e_end) (a multiple of 512 tokens wide, nit blocks) by one
// wave; the result is in every lane.  FAST: 16-byte aligned bf16 rows, four 512-token blocks in flight.
template <bool FAST>
__device__ __forceinline__ double wave_pass_sum(const WalkRows& R, int L, const float* __restrict__ inv_Rf,
                                                int e_begin, int e_end, int nit, int V, float c, int lane) {
  double acc = 0.0;
  if constexpr (FAST) {
    const uint16_t* tp = static_cast<const uint16_t*>(R.t_base) + R.t_off;
    const uint16_t* qp = static_cast<const uint16_t*>(R.q_base) + R.q_off;
    for (int it0 = 0; it0 < nit; it0 += 4) {
      u32x4 rp[4], rq[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e0 = min(e_begin + (it0 + u) * 512 + lane * 8, V - 8);     // clamped; masked below
        rp[u] = *reinterpret_cast<const u32x4*>(tp + e0);
        if (L > 0) rq[u] = *reinterpret_cast<const u32x4*>(qp + e0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int it = it0 + u;
        if (it < nit) {
          const int e0 = e_begin + it * 512 + lane * 8;
          float lp[8], lq[8];
          unpack_bf16x8(rp[u], lp);
          if (L > 0) unpack_bf16x8(rq[u], lq);
          float w[8];
          weights_from(R, lp, lq, e0 < e_end ? 8 : 0, c, L, inv_Rf, w);
          float lsf = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) lsf += w[j];
          acc += static_cast<double>(lsf);
        }
      }
    }
  } else {
    for (int it = 0; it < nit; ++it) {
      const int e0 = e_begin + it * 512 + lane * 8;
      float lsf = 0.f;
      if (e0 < e_end) {
        float w[8];
        weights8(R, e0, V, c, L, inv_Rf, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) lsf += w[j];
      }
      acc += static_cast<double>(lsf);
    }
  }
  return wave_sum(acc);
}

// ---- helper workgroups -----------------------------------------------------------------------
// A full pass over a large vocabulary is bound by the vector ALU of the one compute unit that runs
// the request's walk (two exp2 per class).  For such vocabularies every request gets up to three
// helper workgroups on other compute units: the vocabulary is cut into 16 x (1 + helpers) contiguous
// wave segments, the master publishes what a pass needs, each helper sums its 16 segments and hands
// the sums back, and the master goes on as if it had 64 waves.  The partition is static and the
// grid (masters first, then helpers) is at most one workgroup per compute unit, so every workgroup
// becomes resident without waiting for another; helpers only ever wait for their master, the master
// only for its helpers, and every wait is bounded.
// Everything exchanged goes through relaxed device-scope atomic accesses (they bypass the
// non-coherent cache levels for exactly these words; acquire/release would write back and
// invalidate the whole L2 of the XCD on every poll and evict the logit rows the passes re-read).
// Order between a payload and its flag: the payload's stores have completed (vmcnt 0) before the
// flag is written.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- pieces shared by the kernels that take the scalar accept decisions --------------------------------
// r(x)/q(x) of a drafted token x at residual level 0 from its two logits and the merged row statistics
// (q: a logit, or the probability itself).  q(x) = 0 < p(x) accepts, q(x) = p(x) = 0 rejects.
__device__ __forceinline__ double accept_ratio(double lp, float t_m, double t_invz, double lq, float q_m, double q_invz,
                                               float c, bool q_is_probs) {
  const double px = exp2((lp - static_cast<double>(t_m)) * static_cast<double>(c)) * t_invz;
  const double qx = q_is_probs ? lq : exp2((lq - static_cast<double>(q_m)) * static_cast<double>(c)) * q_invz;
  if (qx > 0.0) return px / qx;
  return (px > 0.0) ? INFINITY : 0.0;
}

// ----------------------------------------------------------------------------------
// Statistics pass for large batches of linear drafts that stops reading a request's rows once its chain is known
// to have ended (Section 2.1: a rejection discards every later token).  Grid (segment, request, level), levels in
// the order the chain needs them: target row 0, then for node j = 0, 1, ... its draft row and target row j + 1.
// The 2 x nseg workgroups that produce the two rows of node j count their arrivals; the last one merges the two
// rows' statistics, gathers the node's two logits and takes the accept decision with the arithmetic the
// linear-draft kernel will use (same functions, same order: same bits); a rejection lowers stop[request] to j.
// A workgroup of a later level looks at stop[request] first and returns without reading when its row lies
// behind the stop.  Workgroups start roughly in grid order, so deep levels usually see the decisions of
// shallow ones; nothing depends on it - whatever was skipped lies behind the final stop, and the linear-draft
// kernel never uses a row behind its own first rejection, which is that same stop.
// ----------------------------------------------------------------------------------
constexpr int kProgMaxNodes = 64;
constexpr int kCntStride = 32;             // ints between two arrival counters: one 128-byte line each
constexpr int kProgStopStride = 32;        // ints between two requests' stop words: one 128-byte line each (every workgroup of a request reads its word)

__global__ __launch_bounds__(kStatThreads) void accept_prog_init_kernel(unsigned* __restrict__ node_cnt, int n_cnt,
                                                                       int* __restrict__ stop, unsigned* __restrict__ arrived, int B) {
  const int t = blockIdx.x * kStatThreads + threadIdx.x, nt = gridDim.x * kStatThreads;
  for (int i = t; i < n_cnt; i += nt) node_cnt[i * kCntStride] = 0u;
  for (int i = t; i < B; i += nt) { stop[i * kProgStopStride] = 0x7fffffff; arrived[i * kCntStride] = 0u; }
}

__global__ __launch_bounds__(kStatThreads) void row_stats_prog_kernel(
    const void* __restrict__ t_base, int t_dtype, int n_t_rows, const void* __restrict__ q_base, int q_dtype, int n_q_rows,
    int V, float c, int nseg, SegStat* __restrict__ stats, const int32_t* __restrict__ node_offsets,
    const int32_t* __restrict__ q_row, const int32_t* __restrict__ draft_tokens, const float* __restrict__ u_accept,
    unsigned* __restrict__ node_cnt, int* __restrict__ stop, int max_nodes) {
  const int seg = blockIdx.x, b = blockIdx.y, k = blockIdx.z;
  const int tid = threadIdx.x;
  // (the three loads are independent: one round trip)
  const int st = ld_dev(stop + b * kProgStopStride);
  const int o = node_offsets[b];
  int n = node_offsets[b + 1] - o;
  n = n < 0 ? 0 : (n > max_nodes ? max_nodes : n);
  const bool is_q = (k & 1) != 0;
  const int j = is_q ? (k - 1) / 2 : k / 2 - 1;          // draft row of node j / target row j + 1 (k = 0: target row 0)
  if (k > 0 && j >= n) return;                           // the request has no such row
  if (k > 0 && (is_q ? st < j : st <= j)) return;        // the chain ended before this row is needed
  const int64_t trow0 = static_cast<int64_t>(o) + b;
  const void* base;
  int dtype;
  int64_t r, srow;
  if (is_q) {
    const int qr = min(max(q_row[o + j], 0), n_q_rows - 1);
    base = q_base; dtype = q_dtype; r = qr; srow = static_cast<int64_t>(n_t_rows) + qr;
  } else {
    base = t_base; dtype = t_dtype; r = trow0 + j + 1; srow = r;
  }
  __shared__ StatScratch sh;
  float M;
  double Z;
  const bool writer = segment_stats(base, dtype, r * static_cast<int64_t>(V), seg * kStatSeg, V, c, sh, M, Z);
  // the node whose decision this row feeds: its own (draft row j) or the one tested against it (target row i: node i)
  const int node = is_q ? j : j + 1;
  if (tid >= kWave) return;           // what is left is one wave's work: the other waves free their slots now
  const int lane = tid;
  int last = 0;
  if (writer) {                       // lane 0
    unsigned long long* w = reinterpret_cast<unsigned long long*>(stats + srow * nseg + seg);
    st_dev(w, static_cast<unsigned long long>(__float_as_uint(M)));
    st_dev(w + 1, __builtin_bit_cast(unsigned long long, Z));
    if (node < n) {
      wait_stores();
      const unsigned old = __hip_atomic_fetch_add(&node_cnt[static_cast<int64_t>(o + node) * kCntStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = (old == static_cast<unsigned>(2 * nseg - 1));
    }
  }
  last = __shfl(last, 0, kWave);
  if (!last) return;
  // ---- both rows of `node` are complete: its accept decision, by this wave ----
  const int x = min(max(draft_tokens[o + node], 0), V - 1);
  const int qr = min(max(q_row[o + node], 0), n_q_rows - 1);
  float m = 0.f;
  double z = 1.0;
  {
    const int which = (lane >> 4) & 1, sl = lane & 15;   // lanes 0-15: the target row, 16-31: the draft row (32-63 repeat them)
    const int64_t sr = which ? static_cast<int64_t>(n_t_rows) + qr : trow0 + node;
    merged_row_stats<true>(stats + sr * nseg, nseg, c, sl, m, z);
  }
  const float m_t = __shfl(m, 0, kWave), m_q = __shfl(m, 16, kWave);
  const double z_t = __shfl(z, 0, kWave), z_q = __shfl(z, 16, kWave);
  if (lane == 0) {
    const double lp = static_cast<double>(load_logit(t_base, t_dtype, (trow0 + node) * static_cast<int64_t>(V) + x));
    const double lq = static_cast<double>(load_logit(q_base, q_dtype, static_cast<int64_t>(qr) * V + x));
    const double ratio = accept_ratio(lp, m_t, 1.0 / z_t, lq, m_q, 1.0 / z_q, c, false);
    if (!(static_cast<double>(u_accept[o + node]) < ratio))
      __hip_atomic_fetch_min(stop + b * kProgStopStride, node, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

constexpr int kMaxHelpers = 3;

// What a helper wave hands back: the sum of its segment and the pass it belongs to.  The wave
// writes the sum, waits for that store to complete, then writes the pass number; the master reads
// the 16 bytes with one load (one access to one cache line), so a matching pass number always comes
// with its sum and a hand-off costs a single trip.
struct __attribute__((aligned(16))) PartSlot {
  double sum;
  unsigned seq;
  unsigned pad;
};
__device__ __forceinline__ PartSlot ld_slot(const PartSlot* p) {
  u32x4 v;
  asm volatile("global_load_dwordx4 %0, %1, off sc0 sc1\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
  PartSlot r;
  r.sum = __builtin_bit_cast(double, (static_cast<unsigned long long>(v[1]) << 32) | v[0]);
  r.seq = v[2];
  r.pad = 0;
  return r;
}
constexpr unsigned kDone = 0xffffffffu;    // pass number that tells the helpers to leave
constexpr int kSpinLimit = 4000;           // a helper whose master never shows up leaves after this many polls (a few
                                           // milliseconds: ten times the master's own patience)

struct PassDesc {            // written by the master, published by `seq` (pass number, from 1)
  unsigned seq;
  int level;
  long long t_off, q_off;
  float t_m, q_m;
  double t_invz, q_invz;
  float inv_R[kMaxNodes];
};

struct AcceptParams {
  int B, V, n_t_rows, n_q_rows, nseg;
  const int32_t* node_offsets;
  const int32_t* parent;
  const int32_t* draft_tokens;
  const void* target; int t_dtype;
  const void* draft_q; int q_dtype; int q_kind;
  const int32_t* q_row;
  float c;                  // log2(e)/T
  const float* u_accept;
  const float* u_resample;
  int32_t* accept_len;
  int32_t* out_tokens; int out_stride;
  int32_t* stop_node;
  float* dbg_ratio;
  const SegStat* stats;
  int helpers;              // helper workgroups per request (0: the master works alone)
  int patience;             // polls a master spends on its helpers before it sums their segments itself
  PassDesc* desc;           // [B]
  PartSlot* part;           // [B][helpers][16] wave sums handed back by the helpers
};

// FAST: 16-byte aligned rows with both logit matrices in bf16 (the default layout): the full
// passes keep four 512-token blocks in flight per wave.
template <bool FAST>
__global__ __launch_bounds__(kWalkThreads) void accept_walk_kernel(AcceptParams P) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int S = P.helpers;
  const int vwaves = kWalkWaves * (1 + S);                 // wave segments the vocabulary is cut into
  __shared__ float sh_inv_Rf[kMaxNodes];     // 1 / R_k, fp32, for the per-class passes
  __shared__ unsigned sh_seq;
  __shared__ int sh_flag;

  // =============================== helper workgroup ===============================
  if (static_cast<int>(blockIdx.x) >= P.B) {
    const int idx = blockIdx.x - P.B;
    const int hb = idx % P.B, h = idx / P.B;               // request, helper number 0..S-1
    const int seg_w = (((P.V + vwaves - 1) / vwaves) + 511) / 512 * 512;
    const int e_begin = ((h + 1) * kWalkWaves + wave) * seg_w;
    const int e_end = min(P.V, e_begin + seg_w);
    const int nit = e_end > e_begin ? (e_end - e_begin + 511) / 512 : 0;
    PassDesc* desc = P.desc + hb;
    unsigned last_seq = 0;
    // Roles inside the loop are per wave, never per lane: with `if (tid == 0)` at the end of one
    // iteration and at the start of the next, the compiler routes the other lanes of wave 0 around
    // both, and they reach the workgroup barrier without lane 0 - a partial wave at s_barrier.
    // All 64 lanes of wave 0 poll (one coalesced load) and store the same words.
    for (;;) {
      if (wave == 0) {
        int spins = 0, fin = 0;
        unsigned seq = 0;
        for (;;) {
          seq = ld_dev(&desc->seq);                          // kDone once the master needs no more passes
          if (seq == kDone) { fin = 1; break; }
          if (seq > last_seq) break;
          __builtin_amdgcn_s_sleep(1);
          if (++spins > kSpinLimit) { fin = 1; break; }      // the master never came: leave
        }
        sh_seq = seq;
        sh_flag = fin;
      }
      __syncthreads();
      if (sh_flag) return;
      const unsigned seq = sh_seq;
      WalkRows R;
      R.t_base = P.target; R.t_dtype = P.t_dtype; R.q_base = P.draft_q; R.q_dtype = P.q_dtype;
      R.q_is_probs = (P.q_kind == 1); R.have_q = 1;
      const int level = ld_dev(&desc->level);
      R.t_off = ld_dev(&desc->t_off); R.q_off = ld_dev(&desc->q_off);
      R.t_m = ld_dev(&desc->t_m); R.q_m = ld_dev(&desc->q_m);
      R.t_invz = ld_dev(&desc->t_invz); R.q_invz = ld_dev(&desc->q_invz);
      sh_inv_Rf[tid & (kMaxNodes - 1)] = ld_dev(&desc->inv_R[tid & (kMaxNodes - 1)]);    // every thread, same values
      __syncthreads();
      // Normally the master rewrites the descriptor only after this helper has handed back the sums of
      // pass `seq`.  A master that ran out of patience may already be at a later pass: the copy above
      // can then mix two passes (every field is still a valid value of one of them, so all reads stay
      // in bounds) and the sum written below carries the old pass number, which the master ignores.
      const double acc = wave_pass_sum<FAST>(R, min(max(level, 0), kMaxNodes), sh_inv_Rf, e_begin, e_end, nit, P.V, P.c, lane);
      PartSlot* slot = P.part + (static_cast<int64_t>(hb) * S + h) * kWalkWaves + wave;
      st_dev(&slot->sum, acc);                   // all lanes of the wave store the same words
      wait_stores();
      st_dev(&slot->seq, seq);
      last_seq = seq;
      __syncthreads();                           // sh_inv_Rf and sh_seq are rewritten in the next round
    }
  }

  // =============================== master workgroup ===============================
  const int b = blockIdx.x;
  const int o = P.node_offsets[b];
  int n = P.node_offsets[b + 1] - o;
  n = n < 0 ? 0 : (n > kMaxNodes ? kMaxNodes : n);
  const int64_t trow0 = static_cast<int64_t>(o) + b;
  const int V = P.V;
  const float c = P.c;
  // contiguous vocab segment of each wave (the master's 16 and the helpers'), a multiple of 512 tokens
  const int seg_w = (((V + vwaves - 1) / vwaves) + 511) / 512 * 512;

  __shared__ double sh_wave_sum[kWalkWaves * (1 + kMaxHelpers)];
  __shared__ unsigned long long sh_missing;
  __shared__ double sh_blk[kMaxBlocksPerSeg];   // sums of the 512-token blocks of the segment the draw falls in
  __shared__ double sh_inv_R[kMaxNodes];     // 1 / R_k for the scalar accept tests
  __shared__ int sh_token;
  // per-request tables filled once, in parallel, so that the walk itself touches no global memory
  __shared__ float sh_tm[kMaxNodes + 1];       // target local row i: max logit
  __shared__ double sh_tinvz[kMaxNodes + 1];   //                     1 / sum 2^((l-m)c)
  __shared__ float sh_qm[kMaxNodes];           // draft row of node j
  __shared__ double sh_qinvz[kMaxNodes];
  __shared__ int sh_par[kMaxNodes], sh_tok[kMaxNodes], sh_qrow[kMaxNodes];
  __shared__ double sh_px[kMaxNodes], sh_qx[kMaxNodes];   // p_parent(x_j), q(x_j)
  __shared__ float sh_u[kMaxNodes];
  __shared__ int sh_fc[kMaxNodes + 1];         // first child (lowest index) of node i at [i + 1]

  const bool q_is_probs = (P.q_kind == 1);
  const double u_res = static_cast<double>(P.u_resample[b]);      // needed last; fetched first
  // (1) node arrays
  if (tid <= kMaxNodes) sh_fc[tid] = kMaxNodes;
  if (tid < n) {
    int par = P.parent ? P.parent[o + tid] : tid - 1;
    if (par < -1 || par >= tid) par = -1;
    sh_par[tid] = par;
    // indices come from device memory the host cannot check: clamp them so that a bad entry
    // gives a wrong answer for that request instead of an out-of-bounds read
    sh_tok[tid] = min(max(P.draft_tokens[o + tid], 0), V - 1);
    sh_qrow[tid] = min(max(P.q_row[o + tid], 0), P.n_q_rows - 1);
    sh_u[tid] = P.u_accept[o + tid];
    if (P.dbg_ratio) P.dbg_ratio[o + tid] = __builtin_nanf("");
  }
  if (tid < kMaxNodes) sh_inv_Rf[tid] = 0.f;
  __syncthreads();
  if (P.parent) {
    // The children of one node were drawn from one draft distribution: the row its first child names.  Every
    // sibling uses that row (for q(x) and for the residual), whatever its own q_row entry says.
    if (tid < n) atomicMin(&sh_fc[sh_par[tid] + 1], tid);
    __syncthreads();
    int group_row = 0;
    if (tid < n) group_row = sh_qrow[min(sh_fc[sh_par[tid] + 1], kMaxNodes - 1)];
    __syncthreads();
    if (tid < n) sh_qrow[tid] = group_row;
    __syncthreads();
  }
  // (2) in one round trip: the two logits of every drafted token (last wave) and the merged
  // statistics of the n+1 target rows and n draft rows (groups of 16 lanes, one segment each)
  if (wave == kWalkWaves - 1) {
    for (int j = lane; j < n; j += kWave) {
      const int x = sh_tok[j];
      sh_px[j] = static_cast<double>(load_logit(P.target, P.t_dtype, (trow0 + 1 + sh_par[j]) * static_cast<int64_t>(V) + x));
      sh_qx[j] = static_cast<double>(load_logit(P.draft_q, P.q_dtype, static_cast<int64_t>(sh_qrow[j]) * V + x));
    }
  } else {
    const int n_rows = (n + 1) + (q_is_probs ? 0 : n);
    const int sl = tid & 15;
    for (int ri = tid >> 4; ri < n_rows; ri += (kWalkThreads - kWave) / 16) {
      const int64_t srow = (ri <= n) ? trow0 + ri : static_cast<int64_t>(P.n_t_rows) + sh_qrow[ri - n - 1];
      float m = -INFINITY;
      for (int sg = sl; sg < P.nseg; sg += 16) m = fmaxf(m, P.stats[srow * P.nseg + sg].m);
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 16));
      double z = 0.0;
      for (int sg = sl; sg < P.nseg; sg += 16) {
        const SegStat st = P.stats[srow * P.nseg + sg];
        if (st.m != -INFINITY) z += st.z * exp2(static_cast<double>(st.m - m) * static_cast<double>(c));
      }
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) z += __shfl_xor(z, d, 16);
      if (sl == 0) {
        if (ri <= n) { sh_tm[ri] = m; sh_tinvz[ri] = 1.0 / z; }
        else { sh_qm[ri - n - 1] = m; sh_qinvz[ri - n - 1] = 1.0 / z; }
      }
    }
  }
  __syncthreads();
  // (3) p(x), q(x) of every node
  if (tid < n) {
    const int par = sh_par[tid];
    sh_px[tid] = exp2((sh_px[tid] - static_cast<double>(sh_tm[par + 1])) * static_cast<double>(c)) * sh_tinvz[par + 1];
    if (!q_is_probs)
      sh_qx[tid] = exp2((sh_qx[tid] - static_cast<double>(sh_qm[tid])) * static_cast<double>(c)) * sh_qinvz[tid];
  }
  __syncthreads();

  // lane l looks after nodes l and l + 64; nodes that do not exist hold an impossible parent
  const int my_parent = (lane < n) ? sh_par[lane] : -2;
  const int my_parent_hi = (lane + kWave < n) ? sh_par[lane + kWave] : -2;

  int cur = -1, depth = 0;
  WalkRows R;
  R.t_base = P.target; R.t_dtype = P.t_dtype;
  R.q_base = P.draft_q; R.q_dtype = P.q_dtype; R.q_is_probs = q_is_probs;
  R.t_off = 0; R.t_m = 0.f; R.t_invz = 0.0;
  R.q_off = 0; R.q_m = 0.f; R.q_invz = 0.0; R.have_q = 0;

  const int e_begin = wave * seg_w;
  const int e_end = min(V, e_begin + seg_w);
  const int nit = e_end > e_begin ? (e_end - e_begin + 511) / 512 : 0;

  // One full pass at residual level L: per-wave sums (the master's and the helpers') to LDS, returns
  // the total.
  unsigned pass_no = 0;
  auto full_pass = [&](int L) -> double {
    __syncthreads();                 // previous readers of the sums are done
    ++pass_no;
    if (S > 0 && wave == 0) {          // all lanes of wave 0 store the same words (no per-lane role, see the helper loop)
      PassDesc* desc = P.desc + b;
      st_dev(&desc->level, L);
      st_dev(&desc->t_off, static_cast<long long>(R.t_off)); st_dev(&desc->q_off, static_cast<long long>(R.q_off));
      st_dev(&desc->t_m, R.t_m); st_dev(&desc->q_m, R.q_m);
      st_dev(&desc->t_invz, R.t_invz); st_dev(&desc->q_invz, R.q_invz);
      for (int k = 0; k < L && k < kMaxNodes; ++k) st_dev(&desc->inv_R[k], sh_inv_Rf[k]);
      wait_stores();
      st_dev(&desc->seq, pass_no);
    }
    const double acc = wave_pass_sum<FAST>(R, L, sh_inv_Rf, e_begin, e_end, nit, V, c, lane);
    if (lane == 0) sh_wave_sum[wave] = acc;
    if (S > 0) {
      if (wave == 0) {               // lane l watches helper wave l (the last one again for lanes beyond)
        const int n_slots = S * kWalkWaves;                     // <= 48
        const int my = min(lane, n_slots - 1);
        const PartSlot* slot = P.part + static_cast<int64_t>(b) * n_slots + my;
        int spins = 0;
        PartSlot got;
        bool up;
        for (;;) {
          got = ld_slot(slot);
          up = got.seq == pass_no;
          if (__all(up)) break;
          if (++spins > P.patience) break;                      // helpers not there (yet): see below
          __builtin_amdgcn_s_sleep(1);
        }
        if (up) sh_wave_sum[kWalkWaves + my] = got.sum;         // lanes beyond n_slots repeat the last slot
        const unsigned long long missing = __ballot(!up) & ((1ull << n_slots) - 1ull);
        if (lane == 0) sh_missing = missing;
      }
      __syncthreads();
      // Segments whose helper wave has not answered within the patience (its workgroup may not be
      // resident yet when other kernels fill the GPU) are summed here instead: the walk never
      // depends on a helper making progress.  A late answer is ignored (its pass number is old).
      unsigned long long miss = sh_missing;
      for (int k = 0; miss; ++k) {
        const int j = __ffsll(static_cast<long long>(miss)) - 1;
        miss &= miss - 1;
        if ((k & (kWalkWaves - 1)) != wave) continue;
        const int hb_begin = (kWalkWaves + j) * seg_w;
        const int hb_end = min(V, hb_begin + seg_w);
        const int hb_nit = hb_end > hb_begin ? (hb_end - hb_begin + 511) / 512 : 0;
        const double a2 = wave_pass_sum<FAST>(R, L, sh_inv_Rf, hb_begin, hb_end, hb_nit, V, c, lane);
        if (lane == 0) sh_wave_sum[kWalkWaves + j] = a2;
      }
    }
    __syncthreads();
    double tot = 0.0;
    for (int w = 0; w < vwaves; ++w) tot += sh_wave_sum[w];
    return tot;
  };

  int level = 0;          // rejections so far at the current node
  int sums_level = -1;    // level whose sums sit in LDS (-1: none)
  double total = 0.0;     // total of those sums

  for (int guard = 0; guard <= kMaxNodes; ++guard) {
    // target row of the current node
    R.t_off = (trow0 + 1 + cur) * static_cast<int64_t>(V);
    R.t_m = sh_tm[cur + 1];
    R.t_invz = sh_tinvz[cur + 1];
    level = 0;
    sums_level = -1;
    R.have_q = 0;

    // children of the current node in index order: two ballot words
    unsigned long long kids = __ballot(my_parent == cur && lane > cur);
    unsigned long long kids_hi = __ballot(my_parent_hi == cur && lane + kWave > cur);
    int accepted = -1;
    while (kids | kids_hi) {
      int ch;
      if (kids) { ch = __ffsll(static_cast<long long>(kids)) - 1; kids &= kids - 1; }
      else { ch = kWave + __ffsll(static_cast<long long>(kids_hi)) - 1; kids_hi &= kids_hi - 1; }
      if (!R.have_q) {
        R.q_off = static_cast<int64_t>(sh_qrow[ch]) * V;
        R.q_m = sh_qm[ch];
        R.q_invz = sh_qinvz[ch];
        R.have_q = 1;
      }
      const double qx = sh_qx[ch];
      double rx = sh_px[ch];
      for (int k = 0; k < level; ++k) {
        double w = rx - qx;
        w = w > 0.0 ? w : 0.0;
        rx = w * sh_inv_R[k];
      }
      double ratio;
      if (qx > 0.0) ratio = rx / qx;
      else ratio = (rx > 0.0) ? INFINITY : 0.0;
      if (P.dbg_ratio && tid == 0) P.dbg_ratio[o + ch] = static_cast<float>(ratio);
      const double u = static_cast<double>(sh_u[ch]);
      if (u < ratio) { accepted = ch; break; }
      // rejected: mass of max(0, r - q)
      const double mass = full_pass(level + 1);
      if (mass > 0.0) {
        __syncthreads();
        if (tid == 0) { sh_inv_R[level] = 1.0 / mass; sh_inv_Rf[level] = static_cast<float>(1.0 / mass); }
        __syncthreads();
        ++level;
        sums_level = level;
        total = mass;
      } else {
        sums_level = -1;           // residual has no mass: r stays as it was
      }
    }
    if (accepted >= 0) {
      if (tid == 0 && depth < P.out_stride) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + depth] = sh_tok[accepted];
      ++depth;
      cur = accepted;
      continue;
    }
    // no child, or every child rejected: draw from the level's weights by inverse CDF
    if (sums_level != level) { total = full_pass(level); sums_level = level; }
    if (S > 0 && wave == 0) st_dev(&P.desc[b].seq, kDone);  // no more passes: the helpers may leave
    const double target = u_res * total;
    int ws = -1;
    double before = 0.0;
    for (int w = 0; w < vwaves; ++w) {
      const double sw = sh_wave_sum[w];
      if (before + sw > target) { ws = w; break; }
      before += sw;
    }
    if (ws < 0) {                    // rounding left no crossing: last wave segment with positive mass
      for (int w = vwaves - 1; w >= 0; --w) if (sh_wave_sum[w] > 0.0) { ws = w; break; }
      if (ws < 0) ws = 0;
      before = 0.0;
      for (int w = 0; w < ws; ++w) before += sh_wave_sum[w];
    }
    // block of 512 tokens inside segment ws: the 16 waves sum its blocks in parallel
    const int ws_begin = ws * seg_w;
    const int ws_end = min(V, ws_begin + seg_w);
    const int ws_nit = ws_end > ws_begin ? (ws_end - ws_begin + 511) / 512 : 0;
    __syncthreads();
    for (int it = wave; it < ws_nit; it += kWalkWaves) {
      const int e0 = ws_begin + it * 512 + lane * 8;
      float lsf = 0.f;
      if (e0 < ws_end) {
        float w[8];
        weights8(R, e0, V, c, level, sh_inv_Rf, w);
#pragma unroll
        for (int j = 0; j < 8; ++j) lsf += w[j];
      }
      const double ls = wave_sum(static_cast<double>(lsf));
      if (lane == 0) sh_blk[it] = ls;
    }
    __syncthreads();
    const double* blk = sh_blk;
    int it_hit = -1;
    double run = before;
    for (int it = 0; it < ws_nit; ++it) {
      const double sblk = blk[it];
      if (run + sblk > target) { it_hit = it; break; }
      run += sblk;
    }
    if (it_hit < 0) {                // rounding: last block of the segment with positive mass
      for (int it = ws_nit - 1; it >= 0; --it) if (blk[it] > 0.0) { it_hit = it; break; }
      if (it_hit < 0) it_hit = 0;
      run = before;
      for (int it = 0; it < it_hit; ++it) run += blk[it];
    }
    if (wave == 0) {
      const int e0 = ws_begin + it_hit * 512 + lane * 8;
      float w[8];
      if (e0 < ws_end) weights8(R, e0, V, c, level, sh_inv_Rf, w);
      else {
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = 0.f;
      }
      float lsf = 0.f;                 // summed exactly as the pass did, so the block sums agree
      int my_last = -1;
#pragma unroll
      for (int j = 0; j < 8; ++j) { lsf += w[j]; if (w[j] > 0.f) my_last = e0 + j; }
      const double ls = static_cast<double>(lsf);
      double inc = ls;                 // inclusive scan of the lane sums
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const double tq = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += tq;
      }
      const unsigned long long cross = __ballot(run + inc > target);
      int found = -1;
      if (cross) {
        const int fl = __ffsll(static_cast<long long>(cross)) - 1;
        // every lane works out its own candidate: no lane-dependent branch ahead of the broadcast
        // (with one, the compiler may let lanes reach the broadcast without the lane they read from)
        int tok = -1;
        double acc = run + inc - ls;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc += static_cast<double>(w[j]);
          if (tok < 0 && acc > target && w[j] > 0.f) tok = e0 + j;
        }
        if (tok < 0) tok = my_last;        // rounding inside the lane: its last positive class
        found = __shfl(tok, fl, kWave);
      }
      if (found < 0) {                     // rounding across lanes: last positive class of the block
        int ml = my_last;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) ml = max(ml, __shfl_xor(ml, d, kWave));
        found = ml >= 0 ? ml : min(V - 1, ws_begin + it_hit * 512);
      }
      if (lane == 0 && depth < P.out_stride) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + depth] = found;
    }
    break;
  }
  if (tid == 0) {
    if (S > 0) st_dev(&P.desc[b].seq, kDone);
    P.accept_len[b] = depth;
    if (P.stop_node) P.stop_node[b] = cur;
  }
  for (int i = depth + 1 + tid; i < P.out_stride; i += kWalkThreads) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + i] = -1;
}

// ----------------------------------------------------------------------------------
// Linear drafts (no parent array): a chain is rejected at most once, so after the scalar accept tests exactly one
// vocabulary-wide distribution is left to draw from - max(0, p - q) of the rejected position, or p after the
// last draft when nothing was rejected (Section 2.1).  accept_linear_kernel spreads that one pass over the chip:
// a unit of one to four 4096-class blocks per workgroup, U workgroups per request.  Every workgroup repeats the
// request's scalar tests (a few dozen values from the row statistics), sums the weights of its blocks and hands
// the block sums over; the workgroup that arrives last adds them, finds the block of the draw and re-reads that
// block alone for the class.  Nobody waits for anybody.
// ----------------------------------------------------------------------------------
constexpr int kLinThreads = 512;
constexpr int kLinWaves = kLinThreads / kWave;
constexpr int kLinBlock = kLinThreads * 8;         // classes one sweep of a workgroup covers
constexpr int kLinMaxBlocks = 4;                   // blocks per unit at most (their loads are issued together)
constexpr int kLinMaxUnits = 512;                  // vocabularies up to 2M classes

// most units a vocabulary can be cut into (one block each): sizes the workspace
int linear_units(int V) { return (V + kLinBlock - 1) / kLinBlock; }

// Classes per workgroup (whole blocks): about two workgroups per compute unit for the whole batch.
static int linear_unit_classes(int B, int V, int n_cu) {
  const int max_units = linear_units(V);
  int U = (2 * n_cu + B - 1) / (B > 0 ? B : 1);
  const int min_units = (max_units + kLinMaxBlocks - 1) / kLinMaxBlocks;
  U = U < min_units ? min_units : (U > max_units ? max_units : U);
  const int per = (V + U - 1) / U;
  return (per + kLinBlock - 1) / kLinBlock * kLinBlock;
}

// Weights of a thread's eight classes in each block of unit k (their loads issued together) and the per-block fp32 sums.
// Identical arithmetic wherever it is called.
template <int TDT, int QDT, int BPU>
__device__ __forceinline__ void unit_weights_from(const WalkRows& R, const Raw8<TDT, BPU>& rp, const Raw8<QDT, BPU>& rq, int k, int L,
                                                  int V, float c, float (&w)[BPU][8], float (&lsf)[BPU]) {
  const float no_scale[1] = {0.f};               // 1/R_k of lower levels: none exist at levels 0 and 1
  const int tid = threadIdx.x;
  auto e0 = [&](int i) { return (k * BPU + i) * kLinBlock + tid * 8; };
#pragma unroll
  for (int i = 0; i < BPU; ++i) {
    lsf[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) w[i][j] = 0.f;
    if ((k * BPU + i) * kLinBlock + __builtin_amdgcn_readfirstlane(tid) * 8 < V) {       // (else none of this wave's classes exist)
      float lp[8], lq[8], x[8];
      take8<false>(R.t_base, R.t_off, e0(i), V, rp, i, lp);
      if (L > 0) take8<false>(R.q_base, R.q_off, e0(i), V, rq, i, lq);
      weights_from(R, lp, lq, 8, c, L, no_scale, x);
      const int first = __any(e0(i) > V - 8) ? e0(i) - first8(e0(i), V) : 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        w[i][j] = j >= first ? x[j] : 0.f;
        lsf[i] += w[i][j];
      }
    }
  }
}

template <int TDT, int QDT, int BPU>
__device__ __forceinline__ void unit_weights(const WalkRows& R, int k, int L, int V, float c, float (&w)[BPU][8], float (&lsf)[BPU]) {
  const int tid = threadIdx.x;
  auto t_off = [&](int) { return R.t_off; };
  auto q_off = [&](int) { return R.q_off; };
  auto e0 = [&](int i) { return (k * BPU + i) * kLinBlock + tid * 8; };
  Raw8<TDT, BPU> rp;
  Raw8<QDT, BPU> rq;
  issue8(R.t_base, t_off, e0, V, rp);
  if (L > 0) issue8(R.q_base, q_off, e0, V, rq);
  unit_weights_from<TDT, QDT, BPU>(R, rp, rq, k, L, V, c, w, lsf);
}

// Per-block totals from the per-thread sums: fp64 across lanes and waves in a fixed order; in every thread.
template <int BPU>
__device__ __forceinline__ void block_totals(const float (&lsf)[BPU], double (&sh_bw)[BPU][kLinWaves], double (&tot)[BPU]) {
  const int wave = threadIdx.x >> 6;
  __syncthreads();                  // earlier readers of sh_bw are done
#pragma unroll
  for (int i = 0; i < BPU; ++i) {
    tot[i] = 0.0;
    sh_bw[i][wave] = wave_sum(static_cast<double>(lsf[i]));      // every lane stores the same value
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < BPU; ++i)
#pragma unroll
    for (int v = 0; v < kLinWaves; ++v) tot[i] += sh_bw[i][v];
}

// Every wave alike: lane l holds the sum of `per` blocks from l * per on (one block up to 262144 classes), scanned;
// returns the total.
__device__ __forceinline__ double scan_blocks(const double* sh_part, int nblocks, double& mine, double& inc_b) {
  const int lane = threadIdx.x & 63, per = (nblocks + kWave - 1) / kWave;
  mine = 0.0;
  for (int k = lane * per; k < min(nblocks, (lane + 1) * per); ++k) mine += sh_part[k];
  inc_b = wave_scan(mine);
  return lane_f64(inc_b, kWave - 1);
}

// Block of the draw: the first whose running sum passes the target (rounding left no crossing: the last with mass), and
// the mass ahead of it.
__device__ __forceinline__ int block_of_draw(const double* sh_part, int nblocks, double mine, double inc_b, double target,
                                             double& before) {
  const int per = (nblocks + kWave - 1) / kWave;
  const unsigned long long hit = __ballot(inc_b > target && mine > 0.0);
  const unsigned long long pos = __ballot(mine > 0.0);
  const int l = hit ? __ffsll(static_cast<long long>(hit)) - 1 : (pos ? 63 - __clzll(static_cast<long long>(pos)) : 0);
  before = 0.0;
  if (l > 0) before = lane_f64(inc_b, l - 1);
  int kb_hit = l * per;
  if (per > 1) {
    int k_pos = kb_hit;
    double run = before, run_pos = before;
    bool found = false;
    for (int k = l * per; k < min(nblocks, (l + 1) * per) && !found; ++k) {
      const double sk = sh_part[k];
      if (sk > 0.0) { k_pos = k; run_pos = run; }
      found = sk > 0.0 && run + sk > target;
      run += sk;
    }
    kb_hit = k_pos;
    before = run_pos;
  }
  return kb_hit;
}

// The class of the draw inside block kb_hit, from this thread's eight weights wh (classes e0 on); the wave it falls in
// writes it.
__device__ __forceinline__ void draw_class(const float (&wh)[8], int e0, int kb_hit, double before, double target, int V,
                                           double* sh_wave, int32_t* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float lsh = 0.f;                    // summed exactly as the block sums were
  int my_last = -1;
#pragma unroll
  for (int j = 0; j < 8; ++j) { lsh += wh[j]; if (wh[j] > 0.f) my_last = e0 + j; }
  const double ls = static_cast<double>(lsh);
  const double inc = wave_scan(ls);   // inclusive scan of the lane sums inside the wave
  __syncthreads();                    // earlier readers of sh_wave are done
  sh_wave[wave] = lane_f64(inc, 63);
  __syncthreads();
  // the wave the crossing falls in (or, when rounding left none, the last one with a positive class) names the class
  int v_hit = -1, v_pos = 0;
  double run = before, acc_w = before;     // mass ahead of this wave; of the wave looked at
#pragma unroll
  for (int v = 0; v < kLinWaves; ++v) {
    const double sv = sh_wave[v];
    if (v == wave) run = acc_w;
    acc_w += sv;
    if (v_hit < 0 && sv > 0.0 && acc_w > target) v_hit = v;
    if (sv > 0.0) v_pos = v;
  }
  if (wave != (v_hit >= 0 ? v_hit : v_pos)) return;
  int found;
  const unsigned long long cross = __ballot(run + inc > target && lsh > 0.f);
  if (cross) {
    // every lane works out its own candidate: no lane-dependent branch ahead of the broadcast
    int tok = -1;
    double acc = run + (inc - ls);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc += static_cast<double>(wh[j]);
      if (tok < 0 && acc > target && wh[j] > 0.f) tok = e0 + j;
    }
    if (tok < 0) tok = my_last;       // rounding inside the lane: its last positive class
    found = __builtin_amdgcn_readlane(tok, __ffsll(static_cast<long long>(cross)) - 1);
  } else {                            // rounding: the last positive class of the wave
    const unsigned long long pos = __ballot(my_last >= 0);
    found = pos ? __builtin_amdgcn_readlane(my_last, 63 - __clzll(static_cast<long long>(pos))) : min(V - 1, kb_hit * kLinBlock);
  }
  if (lane == 0 && out) *out = found;
}

// What bounds it: latency - offsets, node arrays, statistics and logits of the drafted tokens, weights, hand-over,
// block sums, the block of the draw are seven dependent trips to memory at most, so the work between two trips is kept
// short: no barrier between the node arrays and the loads they lead to, every wave takes the accept decisions itself
// (lane j node j, one ballot), reductions and scans run on data-parallel primitives, and the block of the draw is found
// by a scan over the lanes.  Against the version with a barrier per phase and serial searches: 1 request x 1000 classes
// 8.8 -> 5.1 us, 8 x 32000 11.6 -> 8.2, 1 x 128256 13.0 -> 8.5, 64 x 128256 21.1 -> 15.2, 5 x 50257 fp32 16.7 -> 8.2 (one
// element per load before).
//
// BPU: blocks of a unit.  A constant, so that the loads of a unit stand side by side without a branch and are those of its
// own blocks only (with the loads of four blocks whatever their number, the neighbours' read and dropped: 8 x 32000 8.8
// us, 1 x 128256 9.2, 5 x 50257 fp32 9.3; 16 x 128256 with its statistics 21.6 instead of 18.1).
template <int TDT, int QDT, int BPU>
__global__ __launch_bounds__(kLinThreads, 2) void accept_linear_kernel(AcceptParams P, double* __restrict__ partial,
                                                                    unsigned* __restrict__ arrived, int U) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x / U, unit = blockIdx.x % U;
  const int o = P.node_offsets[b];
  int n = P.node_offsets[b + 1] - o;
  n = n < 0 ? 0 : (n > kMaxNodes ? kMaxNodes : n);
  const int64_t trow0 = static_cast<int64_t>(o) + b;
  const int V = P.V;
  __builtin_assume(V >= 8);
  const float c = P.c;
  const bool q_is_probs = (P.q_kind == 1);

  __shared__ float sh_tm[kMaxNodes + 1];
  __shared__ double sh_tinvz[kMaxNodes + 1];
  __shared__ float sh_qm[kMaxNodes];
  __shared__ double sh_qinvz[kMaxNodes];
  __shared__ int sh_tok[kMaxNodes], sh_qrow[kMaxNodes];
  __shared__ float sh_lp[kMaxNodes], sh_lq[kMaxNodes], sh_u[kMaxNodes];
  __shared__ double sh_part[kLinMaxUnits];
  __shared__ int sh_last;
  __shared__ double sh_bw[BPU][kLinWaves];
  const double u_res = static_cast<double>(P.u_resample[b]);
  // (1) the last wave: node arrays (indices clamped: a bad entry gives a wrong answer for that request, never a wild
  // read) and the two logits of every drafted token; the others: the merged statistics of the n+1 target rows and the
  // n draft rows (groups of 16 lanes, one segment each)
  if (wave == kLinWaves - 1) {
    for (int j = lane; j < n; j += kWave) {
      const int x = min(max(P.draft_tokens[o + j], 0), V - 1);
      const int qr = min(max(P.q_row[o + j], 0), P.n_q_rows - 1);
      sh_u[j] = P.u_accept[o + j];
      sh_lp[j] = load_logit(P.target, TDT, (trow0 + j) * static_cast<int64_t>(V) + x);
      sh_lq[j] = load_logit(P.draft_q, QDT, static_cast<int64_t>(qr) * V + x);
      sh_tok[j] = x;
      sh_qrow[j] = qr;
    }
  } else {
    const int n_rows = (n + 1) + (q_is_probs ? 0 : n);
    const int sl = tid & 15;
    for (int r0 = wave * 4; r0 < n_rows; r0 += (kLinThreads - kWave) / 16) {       // (wave-uniform: whole waves reduce)
      const int ri = r0 + (lane >> 4);
      int64_t srow = trow0 + min(ri, n);
      if (ri > n && ri < n_rows) srow = static_cast<int64_t>(P.n_t_rows) + min(max(P.q_row[o + ri - n - 1], 0), P.n_q_rows - 1);
      float m;
      double z;
      merged_row_stats<false>(P.stats + srow * P.nseg, ri < n_rows ? P.nseg : 0, c, sl, m, z);
      if (sl == 0 && ri < n_rows) {
        if (ri <= n) { sh_tm[ri] = m; sh_tinvz[ri] = 1.0 / z; }
        else { sh_qm[ri - n - 1] = m; sh_qinvz[ri - n - 1] = 1.0 / z; }
      }
    }
  }
  __syncthreads();
  // (2) the accept decisions (node j is tested against target row j, the distribution after nodes 0..j-1): lane j of
  // every wave takes nodes j and j + 64, the lowest rejected node ends the chain
  int rejected = -1;
  for (int h = 0; h < n && rejected < 0; h += kWave) {
    const int j = h + lane;
    bool rej = false;
    double ratio = 0.0;
    if (j < n) {
      ratio = accept_ratio(static_cast<double>(sh_lp[j]), sh_tm[j], sh_tinvz[j], static_cast<double>(sh_lq[j]),
                           q_is_probs ? 0.f : sh_qm[j], q_is_probs ? 0.0 : sh_qinvz[j], c, q_is_probs);
      rej = !(static_cast<double>(sh_u[j]) < ratio);
    }
    const unsigned long long rm = __ballot(rej);
    if (rm) rejected = h + __ffsll(static_cast<long long>(rm)) - 1;
    if (unit == 0 && wave == 0 && P.dbg_ratio && j < n)
      P.dbg_ratio[o + j] = (rejected < 0 || j <= rejected) ? static_cast<float>(ratio) : __builtin_nanf("");
  }
  if (unit == 0 && P.dbg_ratio && rejected >= 0)           // nodes of words that were not looked at
    for (int j = (rejected / kWave + 1) * kWave + tid; j < n; j += kLinThreads) P.dbg_ratio[o + j] = __builtin_nanf("");
  const int depth = rejected < 0 ? n : rejected;
  if (unit == 0) {          // everything but the drawn token is known here
    for (int i = tid; i < P.out_stride; i += kLinThreads)
      if (i != depth) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + i] = (i < depth) ? sh_tok[i] : -1;
    if (tid == 0) {
      P.accept_len[b] = depth;
      if (P.stop_node) P.stop_node[b] = depth - 1;
    }
  }
  WalkRows R;
  R.t_base = P.target; R.t_dtype = TDT;
  R.q_base = P.draft_q; R.q_dtype = QDT; R.q_is_probs = q_is_probs;
  R.t_off = (trow0 + depth) * static_cast<int64_t>(V);
  R.t_m = sh_tm[depth]; R.t_invz = sh_tinvz[depth];
  R.have_q = rejected >= 0;
  R.q_off = 0; R.q_m = 0.f; R.q_invz = 0.0;
  int level = 0;
  if (rejected >= 0) {
    R.q_off = static_cast<int64_t>(sh_qrow[rejected]) * V;
    if (!q_is_probs) { R.q_m = sh_qm[rejected]; R.q_invz = sh_qinvz[rejected]; }
    level = 1;
  }

  const int nblocks = (V + kLinBlock - 1) / kLinBlock;
  float w[BPU][8], lsf[BPU];
  double tot[BPU];
  unit_weights<TDT, QDT, BPU>(R, unit, level, V, c, w, lsf);
  block_totals(lsf, sh_bw, tot);
  if (U == 1) {                       // nothing to hand over
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < BPU; ++i)
        if (i < nblocks) sh_part[i] = tot[i];
    }
  } else {
    if (wave == 0) {                  // all lanes of wave 0 store the same words (no per-lane role around barriers)
#pragma unroll
      for (int i = 0; i < BPU; ++i)
        if (unit * BPU + i < nblocks) st_dev(&partial[static_cast<int64_t>(b) * nblocks + unit * BPU + i], tot[i]);
      wait_stores();
      unsigned old = 0;
      if (lane == 0) old = __hip_atomic_fetch_add(&arrived[b * kCntStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      old = __builtin_amdgcn_readfirstlane(old);
      sh_last = (old == static_cast<unsigned>(U - 1));
    }
    __syncthreads();
    if (!sh_last) return;
    // ---- the last workgroup of the request: total, block of the draw, class ----
    for (int k = tid; k < nblocks; k += kLinThreads) sh_part[k] = ld_dev(&partial[static_cast<int64_t>(b) * nblocks + k]);
  }
  __syncthreads();
  double mine, inc_b;
  double total = scan_blocks(sh_part, nblocks, mine, inc_b);
  bool redrawn = false;
  if (level == 1 && !(total > 0.0)) {
    // a residual without mass leaves the distribution as it was: draw from p (sums redone here; rare)
    level = 0;
    R.have_q = 0;
    redrawn = true;
    for (int k = 0; k < U; ++k) {
      unit_weights<TDT, QDT, BPU>(R, k, 0, V, c, w, lsf);
      block_totals(lsf, sh_bw, tot);
      __syncthreads();
      if (tid == 0) {
#pragma unroll
        for (int i = 0; i < BPU; ++i)
          if (k * BPU + i < nblocks) sh_part[k * BPU + i] = tot[i];
      }
    }
    __syncthreads();
    total = scan_blocks(sh_part, nblocks, mine, inc_b);
  }
  const double target = u_res * total;
  double before;
  const int kb_hit = block_of_draw(sh_part, nblocks, mine, inc_b, target, before);
  // that block alone: this thread's eight weights (kept, when the block is of this workgroup's own unit), the wave
  // sums in LDS
  const int e_hit = kb_hit * kLinBlock + tid * 8;
  int e0 = first8(e_hit, V);          // class of wh[0]
  float wh[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) wh[j] = 0.f;
  if (!redrawn && kb_hit / BPU == unit) {
#pragma unroll
    for (int i = 0; i < BPU; ++i)
      if (i == kb_hit - unit * BPU) {
#pragma unroll
        for (int j = 0; j < 8; ++j) wh[j] = w[i][j];
      }
  } else {
    e0 = e_hit;
    const float no_scale[1] = {0.f};
    if (e0 < V) weights8(R, e0, V, c, level, no_scale, wh);
  }
  draw_class(wh, e0, kb_hit, before, target, V, sh_bw[0], depth < P.out_stride ? P.out_tokens + static_cast<int64_t>(b) * P.out_stride + depth : nullptr);
}

template <int TDT, int QDT>
static auto linear_kernel(int blocks) {
  static_assert(kLinMaxBlocks == 4, "one instantiation per number of blocks");
  return blocks == 1 ? accept_linear_kernel<TDT, QDT, 1> : (blocks == 2 ? accept_linear_kernel<TDT, QDT, 2>
       : (blocks == 3 ? accept_linear_kernel<TDT, QDT, 3> : accept_linear_kernel<TDT, QDT, 4>));
}

// ----------------------------------------------------------------------------------
// Linear drafts in one launch: accept_chain_kernel.  A workgroup takes one 8192-class segment of the pair (target row j,
// draft row of node j) of a request, works out the two rows' statistics there and posts them; it gathers those of rows
// 0 .. j, takes the accept decisions itself, and leaves unless the chain ends at node j.  The workgroups of that pair
// still hold its logits: they sum the weights of their segments, post the sums, gather the others', and the one whose
// segment the draw falls into names the class.  Two exchanges instead of a second launch that starts from nothing.
//
// Messages are 64-bit words {data : tag}, relaxed device-scope accesses; the tag is the call's own number, so that the
// workspace needs no clearing (a launch that is being captured is preceded by a kernel that clears them: replays repeat the
// tag; see MessageTag).  Waits are bounded: a workgroup that misses a record after `patience` polls works it out itself, with the same
// arithmetic in the same order, and goes on; nobody's result depends on who came first.  What that costs at worst, every record
// worked out by everybody (patience 0, calls in a loop, us; else 9.5 to 14): 16 x 16 drafts x 8000 classes 41, 8 x 8 x 32000
// 74, 1 x 7 x 128256 256, 1 x 15 x 131072 444.  Beside another stream whose products fill the chip no record was missed for long:
// 293 to 296 us per call, in two launches 296 to 297.
//
// What bounds it: latency.  Offsets, draft row numbers, logits, the two exchanges (a trip each way), the class.
// ----------------------------------------------------------------------------------
constexpr int kChainMaxRecords = 512;      // (nodes + 1) x segments of a request: a thread gathers one
constexpr int kChainBlocks = 2;            // blocks of 4096 classes in a segment
constexpr int kChainWords = 2 * kRecordWords;             // words of a record: (sum, maximum) of the target and of the draft row
constexpr int kChainSumWords = kChainBlocks * kSumWords;  // ... of a segment's weights

struct ChainScratch {
  float m[2][kLinWaves];
  double z[2][kLinWaves];
};

// A thread's share of one segment of the target row [0] and the draft row [1]: exponentials relative to its own maximum m (rows
// whose statistics are taken), or the values as they are.  Classes that do not exist: 0, or -inf.
struct ChainValues {
  float e[2][kChainBlocks][8];
  float m[2];
};

template <bool T, bool Q, int TDT, int QDT>
__device__ __forceinline__ void chain_exponentials(const WalkRows& R, const Raw8<TDT, kChainBlocks>& rt, const Raw8<QDT, kChainBlocks>& rq, int e_seg,
                                                   int V, float c, ChainValues& v, float (&sum)[2]) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    v.m[k] = -INFINITY;
    sum[k] = 0.f;
    if (k == 0 ? !T : !Q) continue;
    float x[kChainBlocks][8];
    auto any = [&](int i) { return e_seg + i * kLinBlock + wave * kWave * 8 < V; };      // this wave has classes of block i
#pragma unroll
    for (int i = 0; i < kChainBlocks; ++i) {
      const int e0 = e_seg + i * kLinBlock + tid * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) x[i][j] = -INFINITY;
      if (any(i)) {
        if (k == 0) take8<false>(R.t_base, R.t_off, e0, V, rt, i, x[i]);
        else take8<false>(R.q_base, R.q_off, e0, V, rq, i, x[i]);
#pragma unroll
        for (int j = 0; j < 8; ++j) v.m[k] = fmaxf(v.m[k], x[i][j]);
      }
    }
    const float mm = (v.m[k] == -INFINITY) ? 0.f : v.m[k];
#pragma unroll
    for (int i = 0; i < kChainBlocks; ++i) {
#pragma unroll
      for (int j = 0; j < 8; ++j) v.e[k][i][j] = 0.f;
      if (any(i))
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          v.e[k][i][j] = fast_exp2((x[i][j] - mm) * c);
          sum[k] += v.e[k][i][j];
        }
    }
  }
}

// (maximum, sum) of every wave's classes of both rows, to LDS.
template <bool T, bool Q>
__device__ __forceinline__ void chain_wave_stats(const ChainValues& v, const float (&sum)[2], float c, ChainScratch& sh) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k == 0 ? !T : !Q) continue;
    const float wm = wave_max(v.m[k]), wmm = (wm == -INFINITY) ? 0.f : wm, mm = (v.m[k] == -INFINITY) ? 0.f : v.m[k];
    double z = static_cast<double>(sum[k]) * static_cast<double>(fast_exp2((mm - wmm) * c));
    if (v.m[k] == -INFINITY) z = 0.0;
    sh.m[k][wave] = wm;               // every lane stores the same value
    sh.z[k][wave] = wave_sum(z);
  }
}

// The thread's weights of a segment at level L and their sums per block.  Exponentials become probabilities by one factor per
// thread and row (fp64 up to its rounding); values as they are by an exponential each (target) or as probabilities (draft).
template <bool T, bool Q, int TDT, int QDT>
__device__ __forceinline__ void chain_weights(const WalkRows& R, const ChainValues& v, const Raw8<TDT, kChainBlocks>& rt,
                                              const Raw8<QDT, kChainBlocks>& rq, int seg, int L, int V, float c, float (&w)[kChainBlocks][8],
                                              float (&lsf)[kChainBlocks]) {
  const int tid = threadIdx.x;
  float f[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k == 0 ? !T : (!Q || L == 0)) continue;
    // (a thread without a finite logit has exponentials 0 and takes the row's maximum for its own: a factor from any fixed number
    // overflows where the row lies far below it, and 0 x inf is no weight.  A row of -inf throughout stays NaN)
    const float row_m = k ? R.q_m : R.t_m, mm = (v.m[k] == -INFINITY) ? row_m : v.m[k];
    f[k] = static_cast<float>(exp2(static_cast<double>(mm - row_m) * static_cast<double>(c)) * (k ? R.q_invz : R.t_invz));
  }
  const float t_invz = static_cast<float>(R.t_invz);
#pragma unroll
  for (int i = 0; i < kChainBlocks; ++i) {
    const int e0 = seg * kChainBlocks * kLinBlock + i * kLinBlock + tid * 8;
    lsf[i] = 0.f;
    float lp[8], lq[8];
    if constexpr (!T) take8<false>(R.t_base, R.t_off, e0, V, rt, i, lp);
    if constexpr (!Q) {
      if (L > 0) take8<false>(R.q_base, R.q_off, e0, V, rq, i, lq);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float p, q = 0.f;
      if constexpr (T) p = v.e[0][i][j] * f[0];
      else p = fast_exp2((lp[j] - R.t_m) * c) * t_invz;
      if (L > 0) {
        if constexpr (Q) q = v.e[1][i][j] * f[1];
        else q = lq[j] == -INFINITY ? 0.f : lq[j];
        p = fmaxf(p - q, 0.f);
      }
      w[i][j] = p;
      lsf[i] += p;
    }
  }
}

// T_STATS: the statistics of the target rows are taken here (else they lie in P.stats); Q_STATS: draft rows are logits.
template <int TDT, int QDT, bool T_STATS, bool Q_STATS>
__global__ __launch_bounds__(kLinThreads, 4) void accept_chain_kernel(AcceptParams P, unsigned long long* __restrict__ msg,
                                                                      unsigned long long* __restrict__ sums, unsigned long long tag, int levels) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int S = P.nseg, V = P.V;
  const int seg = blockIdx.x % S, bj = blockIdx.x / S, j = bj % levels, b = bj / levels;
  const int o = P.node_offsets[b];
  int n = P.node_offsets[b + 1] - o;
  n = n < 0 ? 0 : min(n, levels - 1);
  if (j > n) return;
  const int64_t trow0 = static_cast<int64_t>(o) + b;
  __builtin_assume(V >= 8);
  const float c = P.c;
  constexpr bool q_is_probs = !Q_STATS;

  __shared__ float sh_m[2][kChainMaxRecords];
  __shared__ double sh_z[2][kChainMaxRecords];
  __shared__ unsigned char sh_have[kChainMaxRecords];
  __shared__ float sh_tm[kMaxNodes + 1], sh_qm[kMaxNodes];
  __shared__ double sh_tinvz[kMaxNodes + 1], sh_qinvz[kMaxNodes];
  __shared__ int sh_tok[kMaxNodes], sh_qrow[kMaxNodes];
  __shared__ float sh_lp[kMaxNodes], sh_lq[kMaxNodes], sh_u[kMaxNodes];
  __shared__ double sh_part[kChainMaxRecords];
  __shared__ double sh_bw[kChainBlocks][kLinWaves];
  __shared__ ChainScratch sh_stat;

  // ---- this workgroup's logits, and (last wave) the node arrays with the two logits of every drafted token ----
  WalkRows R;
  R.t_base = P.target; R.t_dtype = TDT;
  R.q_base = P.draft_q; R.q_dtype = QDT; R.q_is_probs = q_is_probs;
  R.t_off = (trow0 + j) * static_cast<int64_t>(V);
  R.q_off = 0; R.q_m = 0.f; R.q_invz = 0.0;
  R.have_q = 0;
  auto q_off_of = [&](int i) { return static_cast<int64_t>(min(max(P.q_row[o + i], 0), P.n_q_rows - 1)) * V; };
  auto e_of = [&](int sg) { return [=](int i) { return sg * kChainBlocks * kLinBlock + i * kLinBlock + tid * 8; }; };
  Raw8<TDT, kChainBlocks> rt;
  Raw8<QDT, kChainBlocks> rq;
  if constexpr (T_STATS) issue8(R.t_base, [&](int) { return R.t_off; }, e_of(seg), V, rt);
  const bool tested = j < n;          // row j has a draft row
  const double u_res = static_cast<double>(P.u_resample[b]);
  if (tested) R.q_off = q_off_of(j);
  if constexpr (Q_STATS) issue8(R.q_base, [&](int) { return R.q_off; }, e_of(seg), V, rq);      // (row n: draft row 0, unused)
  const int n_seen = min(j + 1, n);   // nodes whose decisions this workgroup takes
  if (wave == kLinWaves - 1) {
    for (int i = lane; i < n_seen; i += kWave) {
      const int x = min(max(P.draft_tokens[o + i], 0), V - 1);
      const int qr = min(max(P.q_row[o + i], 0), P.n_q_rows - 1);
      sh_u[i] = P.u_accept[o + i];
      sh_lp[i] = load_logit(P.target, TDT, (trow0 + i) * static_cast<int64_t>(V) + x);
      sh_lq[i] = load_logit(P.draft_q, QDT, static_cast<int64_t>(qr) * V + x);
      sh_tok[i] = x;
      sh_qrow[i] = qr;
    }
  }
  const int n_rec = (j + 1) * S, own = j * S + seg;
  if constexpr (!T_STATS) {
    if (tid < n_rec) {
      const SegStat st = P.stats[trow0 * S + tid];
      sh_m[0][tid] = st.m; sh_z[0][tid] = st.z;
    }
    if constexpr (!Q_STATS) __syncthreads();
  }
  ChainValues val;
  // ... of another segment or pair, from memory (records and sums that did not come)
  auto values_of = [&](const WalkRows& X, int sg, int L, Raw8<TDT, kChainBlocks>& xt, Raw8<QDT, kChainBlocks>& xq, ChainValues& v,
                       float (&sum)[2]) __attribute__((always_inline)) {
    issue8(X.t_base, [&](int) { return X.t_off; }, e_of(sg), V, xt);
    if (L > 0) issue8(X.q_base, [&](int) { return X.q_off; }, e_of(sg), V, xq);
    chain_exponentials<T_STATS, Q_STATS>(X, xt, xq, sg * kChainBlocks * kLinBlock, V, c, v, sum);
  };
  if constexpr (T_STATS || Q_STATS) {
    float sum[2];
    chain_exponentials<T_STATS, Q_STATS>(R, rt, rq, seg * kChainBlocks * kLinBlock, V, c, val, sum);
    chain_wave_stats<T_STATS, Q_STATS>(val, sum, c, sh_stat);
    __syncthreads();
    unsigned long long* to = msg + ((trow0 + j) * S + seg) * kChainWords;
    if constexpr (T_STATS) {          // a thread per word: the target row's record, then the draft row's
      const int kind = tid / kRecordWords;
      if (tid < kChainWords && (kind == 0 || Q_STATS)) {
        float M;
        double Z;
        merge_waves<kLinWaves>(sh_stat.m[kind], sh_stat.z[kind], c, M, Z);
        if (tid % kRecordWords == 0) { sh_m[kind][own] = M; sh_z[kind][own] = Z; }
        st_dev(to + tid, message_word(tid % kRecordWords, Z, M, tag));
      }
    } else if (tid == 0) {            // the draft row's alone, by one thread (by a thread per word 2 x 3 drafts x 3968 classes 9.9 us instead of 9.7)
      float M;
      double Z;
      merge_waves<kLinWaves>(sh_stat.m[1], sh_stat.z[1], c, M, Z);
      sh_m[1][own] = M; sh_z[1][own] = Z;
#pragma unroll
      for (int k = 0; k < record_words(QDT); ++k) st_dev(to + kRecordWords + k, message_word(k, Z, M, tag));
    }
    // ---- gather: thread r the record of segment r % S of rows r / S ----
    bool have = true;
    if (tid < (n_rec + kWave - 1) / kWave * kWave) {            // (wave-uniform)
      const bool mine = tid < n_rec && tid != own;
      const int i = tid / S, sg = tid - i * S;
      const unsigned long long* from = msg + ((trow0 + min(i, j)) * S + sg) * kChainWords;
      const bool want_q = Q_STATS && i < n;
      unsigned long long w[kChainWords];
#pragma unroll
      for (int k = 0; k < kChainWords; ++k) w[k] = 0ull;
      for (int poll = 0;; ++poll) {
        have = true;
        if (mine) {
#pragma unroll
          for (int k = 0; k < kChainWords; ++k)
            if (k < kRecordWords ? T_STATS && k < record_words(TDT) : Q_STATS && k - kRecordWords < record_words(QDT)) w[k] = ld_dev(from + k);
          if constexpr (T_STATS) have = have_tag<record_words(TDT)>(w, tag);
          if constexpr (Q_STATS) have &= !want_q || have_tag<record_words(QDT)>(w + kRecordWords, tag);
        }
        if (__all(have) || poll >= P.patience) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (tid < n_rec) {
        sh_have[tid] = have;
        if (tid != own) {
          if constexpr (T_STATS) { sh_m[0][tid] = message_max<record_words(TDT)>(w); sh_z[0][tid] = message_sum(w); }
          if constexpr (Q_STATS) { sh_m[1][tid] = message_max<record_words(QDT)>(w + kRecordWords); sh_z[1][tid] = message_sum(w + kRecordWords); }
        }
      }
    }
    if (__syncthreads_or(!have)) {    // records that did not come: worked out here
      for (int r = 0; r < n_rec; ++r) {
        if (sh_have[r]) continue;
        const int i = r / S, sg = r % S;
        WalkRows X = R;
        X.t_off = (trow0 + i) * static_cast<int64_t>(V);
        X.q_off = i < n ? q_off_of(i) : 0;
        Raw8<TDT, kChainBlocks> xt;
        Raw8<QDT, kChainBlocks> xq;
        ChainValues v;
        values_of(X, sg, Q_STATS, xt, xq, v, sum);
        __syncthreads();              // earlier readers of sh_stat are done
        chain_wave_stats<T_STATS, Q_STATS>(v, sum, c, sh_stat);
        __syncthreads();
        if (tid < 2 && (tid == 0 ? T_STATS : Q_STATS)) merge_waves<kLinWaves>(sh_stat.m[tid], sh_stat.z[tid], c, sh_m[tid][r], sh_z[tid][r]);
      }
      __syncthreads();
    }
  }
  // ---- merged statistics of target rows 0 .. j and of the draft rows tested against them ----
  {
    const int n_rows = (j + 1) + (Q_STATS ? n_seen : 0);
    const int sl = tid & 15;
    for (int r0 = wave * 4; r0 < n_rows; r0 += kLinThreads / 16) {                 // (wave-uniform: whole waves reduce)
      const int ri = r0 + (lane >> 4);
      const bool is_q = ri > j, any = ri < n_rows;
      const int i = is_q ? ri - (j + 1) : ri;
      float m;
      double z;
      merged_stats([&](int sg) -> SegStat {
        SegStat st;
        st.m = sh_m[is_q][i * S + sg]; st.pad = 0.f; st.z = sh_z[is_q][i * S + sg];
        return st;
      }, any ? S : 0, c, sl, m, z);
      if (sl == 0 && any) {
        if (is_q) { sh_qm[i] = m; sh_qinvz[i] = 1.0 / z; }
        else { sh_tm[i] = m; sh_tinvz[i] = 1.0 / z; }
      }
    }
  }
  __syncthreads();
  // ---- the accept decisions on nodes 0 .. j, by every wave (lane i nodes i, i + 64): the chain ends here or not ----
  auto ratio_of = [&](int i) {
    return accept_ratio(static_cast<double>(sh_lp[i]), sh_tm[i], sh_tinvz[i], static_cast<double>(sh_lq[i]),
                        q_is_probs ? 0.f : sh_qm[i], q_is_probs ? 0.0 : sh_qinvz[i], c, q_is_probs);
  };
  int rejected = -1;
  for (int h = 0; h < n_seen && rejected < 0; h += kWave) {
    const int i = h + lane;
    bool rej = false;
    if (i < n_seen) rej = !(static_cast<double>(sh_u[i]) < ratio_of(i));
    const unsigned long long rm = __ballot(rej);
    if (rm) rejected = h + __ffsll(static_cast<long long>(rm)) - 1;
  }
  if (rejected >= 0 ? rejected < j : j < n) return;
  const int depth = j;
  if (seg == 0) {           // everything but the drawn token is known here
    if (P.dbg_ratio) {
      for (int i = tid; i < n; i += kLinThreads) P.dbg_ratio[o + i] = i <= depth ? static_cast<float>(ratio_of(i)) : __builtin_nanf("");
    }
    for (int i = tid; i < P.out_stride; i += kLinThreads)
      if (i != depth) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + i] = (i < depth) ? sh_tok[i] : -1;
    if (tid == 0) {
      P.accept_len[b] = depth;
      if (P.stop_node) P.stop_node[b] = depth - 1;
    }
  }
  int level = rejected >= 0;
  R.t_m = sh_tm[depth]; R.t_invz = sh_tinvz[depth];
  R.have_q = level;
  if (Q_STATS && level) { R.q_m = sh_qm[depth]; R.q_invz = sh_qinvz[depth]; }
  if constexpr (!T_STATS) issue8(R.t_base, [&](int) { return R.t_off; }, e_of(seg), V, rt);
  if constexpr (!Q_STATS)
    if (level) issue8(R.q_base, [&](int) { return R.q_off; }, e_of(seg), V, rq);

  // ---- weights of this segment, the sums of all segments ----
  const int nblocks = (V + kLinBlock - 1) / kLinBlock;
  float w[kChainBlocks][8], lsf[kChainBlocks];
  double tot[kChainBlocks];
  chain_weights<T_STATS, Q_STATS>(R, val, rt, rq, seg, level, V, c, w, lsf);
  block_totals(lsf, sh_bw, tot);
  // ... of another segment of this pair, from memory
  auto weights_of = [&](int k, int L, float (&wx)[kChainBlocks][8], float (&lx)[kChainBlocks], double (&tx)[kChainBlocks]) {
    Raw8<TDT, kChainBlocks> xt;
    Raw8<QDT, kChainBlocks> xq;
    ChainValues v;
    float sum[2];
    values_of(R, k, L, xt, xq, v, sum);
    chain_weights<T_STATS, Q_STATS>(R, v, xt, xq, k, L, V, c, wx, lx);
    block_totals(lx, sh_bw, tx);
  };
  if (S > 1) {
    unsigned long long* mine = sums + static_cast<int64_t>(b) * S * kChainSumWords;
    if (wave == 0 && lane < kChainSumWords) {
      const int i = lane >= kSumWords;
      st_dev(mine + seg * kChainSumWords + lane, message_word(lane - i * kSumWords, i ? tot[1] : tot[0], 0.f, tag));
    }
    bool have = true;
    if (tid < (nblocks + kWave - 1) / kWave * kWave) {          // (wave-uniform) thread k gathers block k
      const bool want = tid < nblocks && tid / kChainBlocks != seg;
      unsigned long long w[kSumWords] = {0ull, 0ull, 0ull};
      for (int poll = 0;; ++poll) {
        have = true;
        if (want) {
#pragma unroll
          for (int k = 0; k < kSumWords; ++k) w[k] = ld_dev(mine + tid * kSumWords + k);
          have = have_tag<kSumWords>(w, tag);
        }
        if (__all(have) || poll >= P.patience) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (tid < nblocks) {
        sh_have[tid] = have;
        sh_part[tid] = want ? message_sum(w) : (tid & 1 ? tot[1] : tot[0]);
      }
    }
    if (__syncthreads_or(!have)) {
      float wx[kChainBlocks][8], lx[kChainBlocks];
      double tx[kChainBlocks];
      for (int k = 0; k < S; ++k) {
        if (sh_have[k * kChainBlocks] && (k * kChainBlocks + 1 >= nblocks || sh_have[k * kChainBlocks + 1])) continue;
        weights_of(k, level, wx, lx, tx);
        if (tid == 0) {
#pragma unroll
          for (int i = 0; i < kChainBlocks; ++i)
            if (k * kChainBlocks + i < nblocks) sh_part[k * kChainBlocks + i] = tx[i];
        }
      }
    }
  } else if (tid == 0) {
#pragma unroll
    for (int i = 0; i < kChainBlocks; ++i)
      if (i < nblocks) sh_part[i] = tot[i];
  }
  __syncthreads();
  double mine, inc_b;
  double total = scan_blocks(sh_part, nblocks, mine, inc_b);
  bool redrawn = false;
  if (level == 1 && !(total > 0.0)) {
    // a residual without mass leaves the distribution as it was: draw from p (one workgroup alone; rare)
    if (seg != 0) return;
    level = 0;
    redrawn = true;
    __syncthreads();                  // earlier readers of sh_part are done
    for (int k = 0; k < S; ++k) {
      weights_of(k, 0, w, lsf, tot);
      if (tid == 0) {
#pragma unroll
        for (int i = 0; i < kChainBlocks; ++i)
          if (k * kChainBlocks + i < nblocks) sh_part[k * kChainBlocks + i] = tot[i];
      }
    }
    __syncthreads();
    total = scan_blocks(sh_part, nblocks, mine, inc_b);
  }
  const double target = u_res * total;
  double before;
  const int kb_hit = block_of_draw(sh_part, nblocks, mine, inc_b, target, before);
  if (redrawn) weights_of(kb_hit / kChainBlocks, 0, w, lsf, tot);
  else if (kb_hit / kChainBlocks != seg) return;    // (the same for all workgroups of the pair: one stays)
  float wh[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) wh[i] = kb_hit & 1 ? w[1][i] : w[0][i];
  draw_class(wh, first8(kb_hit * kLinBlock + tid * 8, V), kb_hit, before, target, V, sh_bw[0],
             depth < P.out_stride ? P.out_tokens + static_cast<int64_t>(b) * P.out_stride + depth : nullptr);
}

// Workspace: [row statistics][helper protocol: pass descriptors, hand-back slots (zeroed by the
// statistics kernel)]
struct AcceptLayout {
  size_t words_off, n_zero_words, desc_off, part_off, arrived_off, msg_off, lin_off, prog_cnt_off, prog_stop_off, total;
};

static AcceptLayout accept_layout(int B, int total_nodes, int n_q_rows, int V) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  AcceptLayout l;
  const size_t rows = static_cast<size_t>(total_nodes) + B + n_q_rows;
  l.words_off = up(rows * stats_segments(V) * sizeof(SegStat));
  l.desc_off = l.words_off;
  l.part_off = l.desc_off + up(static_cast<size_t>(B) * sizeof(PassDesc));
  l.arrived_off = l.part_off + up(static_cast<size_t>(B) * kMaxHelpers * kWalkWaves * sizeof(PartSlot));
  l.msg_off = l.arrived_off + up(static_cast<size_t>(B) * kCntStride * sizeof(unsigned));   // arrival counters of the linear-draft kernel
  l.n_zero_words = (l.msg_off - l.words_off) / sizeof(unsigned);         // flags, descriptors, hand-back slots, counters
  l.lin_off = l.msg_off + up(cluster_msg_bytes(B));                      // messages of the cluster path
  l.prog_cnt_off = l.lin_off + up(static_cast<size_t>(B) * linear_units(V) * sizeof(double));   // block sums of the linear-draft kernel
  l.prog_stop_off = l.prog_cnt_off + up(static_cast<size_t>(total_nodes) * kCntStride * sizeof(unsigned));   // arrivals per node
  l.total = l.prog_stop_off + up(static_cast<size_t>(B) * kProgStopStride * sizeof(int)) + 256;      // first rejection per request
  return l;
}

size_t accept_workspace_bytes(int B, int total_nodes, int n_q_rows, int V) {
  return accept_layout(B, total_nodes, n_q_rows, V).total;
}

// Where the cluster path wins (measured): every 8192-logit unit of a row gets a compute unit of its own and
// the rows are long.  Short rows and batches with few compute units per request are faster through the
// statistics pass over all rows, whose arithmetic spreads over the whole chip.
static bool cluster_pays(int B, int V, int n_cu) {
  const int units = (V + 8191) / 8192;
  return units >= 8 && units <= 32 && static_cast<int64_t>(B) * units <= n_cu;
}

// Linear drafts take the statistics pass and accept_linear_kernel unless the caller asks for another path (a
// vocabulary of fewer classes than one 16-byte load stays with the walk kernel).
static bool linear_path(const AcceptArgs& a) {
  return a.parent == nullptr && a.V >= 8 && (a.path == 0 || a.path == 3 || a.path == 4) && linear_units(a.V) <= kLinMaxUnits;
}

// Where the one-launch kernel takes a linear draft: one thread gathers one record, the messages lie behind the target
// statistics a caller supplies, and the launch is small.
static size_t chain_offset(const AcceptArgs& a) {
  return a.target_stats_ready ? (static_cast<size_t>(a.total_nodes + a.B) * stats_segments(a.V) * sizeof(SegStat) + 255) / 256 * 256 : 0;
}
static size_t chain_words(const AcceptArgs& a) {
  return static_cast<size_t>(stats_segments(a.V)) * (static_cast<size_t>(a.total_nodes + a.B) * kChainWords + static_cast<size_t>(a.B) * kChainSumWords);
}
// The line: up to five workgroups with rows per four compute units and 48 KB of logits per compute unit.  Beyond, workgroups that wait
// share their units with others that work and the two launches are the faster.  Kernel times (the two launches have the
// gap between them, 1 to 1.5 us, on top), chain / statistics + draw: 1 x 2 drafts x 1000 classes 7.8 / 8.6, 48 x 4 x
// 2000 9.0 / 11.0, 16 x 16 x 8000 11.1 / 13.2, 4 x 8 x 32000 fp32 11.1 / 12.4, 8 x 8 x 32000 11.7 / 13.4, 32 x 4 x 16000 (320
// workgroups) 13.2 / 13.5; 12 x 8 x 32000 (432) 13.2 / 13.7 but slower in a step, 3 x 8 x 128256 (432) 13.5 / 13.2, 16 x 8 x
// 32000 (576) 17.4 / 14.5, 8 x 8 x 32000 fp32 (18 MB) 13.7 / 13.6, 5 x 3 to 9 x 50257 fp32 (245, 14 MB) 13.5 / 13.3 and 1 % behind
// in a step; ragged drafts, calls in a loop: 12 x 1 to 10 x 32000 12.9 / 13.3, 30 x 1 to 16 x 8000 11.8 / 12.9.
// And where workgroups share units, the more segments a row has the more there is to gather, while the grid's places for levels
// that a request does not have cost a little each.  Steps of attention and acceptance, workgroups / grid, chain / two launches (us),
// rows of up to two segments: 274 / 336 24.0 / 25.4, 255 / 2040 26.2 / 29.0; three and four: 270 / 270 26.4 / 27.8, 276 / 352 36.0 /
// 36.1, 248 / 440 22.9 / 22.5, 204 / 1224 19.2 / 19.0; more: 230 / 270 22.3 / 23.0, 216 / 288 25.4 / 25.5, 253 / 330 25.3 / 24.5, 288
// / 432 25.9 / 25.1, 308 / 308 28.4 / 27.6.
static bool chain_path(const AcceptArgs& a) {
  if (!linear_path(a) || a.path != 0 || a.max_nodes > kMaxNodes) return false;
  const int64_t S = stats_segments(a.V), levels = a.max_nodes + 1, n_cu = current_device_cus();
  if (levels * S > kChainMaxRecords || S * kChainBlocks > kChainMaxRecords) return false;
  const int64_t rows = static_cast<int64_t>(a.total_nodes) + a.B;       // (workgroups of levels that a request does not have leave at once)
  const int64_t wgs = rows * S, grid = levels * S * a.B;
  if (wgs * 4 > n_cu * 5 || grid > n_cu * 8) return false;
  if (S > 2 && (wgs + grid) * 2 > n_cu * (S > 4 ? 4 : 5)) return false;
  if (rows * a.V * ((a.t_dtype == kBF16 ? 2 : 4) + (a.q_dtype == kBF16 ? 2 : 4)) > n_cu * 49152) return false;
  return chain_offset(a) + chain_words(a) * sizeof(unsigned long long) <= accept_layout(a.B, a.total_nodes, a.n_q_rows, a.V).total;
}

// The statistics pass that stops at each request's first rejection pays when the launch is several times what
// the chip holds at once (about 2048 workgroups): later levels then start after the decisions of earlier ones.
// The line (workgroups over all rows; whole calls, first rejections / all rows, us): 6528 32.4 / 29.4, 7200 41.2 / 37.9, 8448 40.1
// / 37.9, 9216 43.1 / 41.3; 10752 41.5 / 42.2, 10880 40.6 / 43.8, 12800 39.7 / 48.2, 14784 42.9 / 48.9.
// It needs draft logits (their statistics are part of the decision) and computes the target rows itself.
static bool progressive_stats(const AcceptArgs& a) {
  if (!linear_path(a) || a.q_kind != 0 || a.target_stats_ready || a.total_nodes <= 0) return false;
  if (a.max_nodes > kProgMaxNodes || a.B > 65535) return false;
  const int64_t wgs = (static_cast<int64_t>(a.total_nodes) * 2 + a.B) * stats_segments(a.V);
  return a.path == 4 || (a.path == 0 && wgs >= 9728);
}

const char* accept_plan_name(const AcceptArgs& a, int n_cu) {
  const bool vec = (a.V % 8 == 0) && aligned16(a.target) && aligned16(a.draft_q);
  const bool cluster_ok = vec && a.V >= 8 && a.V <= kClusterMaxV && a.t_dtype == kBF16 && a.q_dtype == kBF16 &&
                          a.q_kind == 0;
  const bool cluster = cluster_ok && (a.path == 2 || (a.path == 0 && a.parent != nullptr && cluster_pays(a.B, a.V, n_cu)));
  if (!cluster && chain_path(a)) return "accept_chain_kernel (one launch in place of row_stats_kernel + accept_linear_kernel: a vocabulary segment of one row pair per workgroup)";
  if (!cluster && progressive_stats(a)) return "row_stats_prog_kernel (rows up to each request's first rejection) + accept_linear_kernel (linear drafts: one vocabulary unit per workgroup, the last to arrive draws)";
  if (!cluster && linear_path(a)) return "row_stats_kernel (all rows) + accept_linear_kernel (linear drafts: one vocabulary unit per workgroup, the last to arrive draws)";
  if (!cluster) return "row_stats_kernel (all rows) + accept_walk_kernel (one workgroup per request, helper workgroups)";
  const ClusterPlan p = make_cluster_plan(a.B, a.V, a.max_nodes, a.parent != nullptr, n_cu, a.levels, a.slices);
  return p.solo ? "accept_cluster_kernel (one workgroup per request, rows of the walked path only)"
                : "accept_cluster_kernel (cluster of workgroups per request, row slices held in registers or LDS)";
}

// Draft rows whose statistics count.  Without nodes nothing was drawn from any: whatever is handed in (a null pointer
// among it) is not read, every request draws from its one target row, and no launch of a row per node is empty.
static int draft_stat_rows(const AcceptArgs& a) { return a.q_kind == 0 && a.total_nodes > 0 ? a.n_q_rows : 0; }

static AcceptParams accept_params(const AcceptArgs& a, int n_t_rows, float c, const SegStat* stats) {
  AcceptParams P;
  P.B = a.B; P.V = a.V; P.n_t_rows = n_t_rows; P.n_q_rows = a.n_q_rows > 0 ? a.n_q_rows : 1; P.nseg = stats_segments(a.V);
  P.node_offsets = a.node_offsets; P.parent = a.parent; P.draft_tokens = a.draft_tokens;
  P.target = a.target; P.t_dtype = a.t_dtype;
  P.draft_q = a.draft_q; P.q_dtype = a.q_dtype; P.q_kind = a.q_kind;
  P.q_row = a.q_row; P.c = c; P.u_accept = a.u_accept; P.u_resample = a.u_resample;
  P.accept_len = a.accept_len; P.out_tokens = a.out_tokens; P.out_stride = a.out_stride;
  P.stop_node = a.stop_node; P.dbg_ratio = a.dbg_ratio; P.stats = stats;
  P.helpers = 0; P.patience = 0; P.desc = nullptr; P.part = nullptr;
  return P;
}

template <int TDT, int QDT>
static auto chain_kernel(const AcceptArgs& a) {
  const bool q_stats = draft_stat_rows(a) > 0;
  return a.target_stats_ready ? (q_stats ? accept_chain_kernel<TDT, QDT, false, true> : accept_chain_kernel<TDT, QDT, false, false>)
                              : (q_stats ? accept_chain_kernel<TDT, QDT, true, true> : accept_chain_kernel<TDT, QDT, true, false>);
}

void launch_accept(const AcceptArgs& a, hipStream_t stream) {
  if (a.B <= 0) return;
  const float c = kLog2e / a.temperature;
  const int n_t_rows = a.total_nodes + a.B;
  const int n_q_stat_rows = draft_stat_rows(a);
  const AcceptLayout lay = accept_layout(a.B, a.total_nodes, a.n_q_rows, a.V);
  unsigned char* ws = static_cast<unsigned char*>(a.workspace);
  const int n_cu = current_device_cus();
  {
    // bf16 logit rows (the default layout): one kernel that reads only the rows the walk reaches (it takes the
    // statistics of those rows itself; target statistics a caller supplies are not needed then)
    const bool vec0 = (a.V % 8 == 0) && aligned16(a.target) && aligned16(a.draft_q);
    const bool cluster_ok = vec0 && a.V >= 8 && a.V <= kClusterMaxV && a.t_dtype == kBF16 && a.q_dtype == kBF16 &&
                            a.q_kind == 0;
    if (cluster_ok && (a.path == 2 || (a.path == 0 && a.parent != nullptr && cluster_pays(a.B, a.V, n_cu)))) {
      const ClusterPlan plan = make_cluster_plan(a.B, a.V, a.max_nodes, a.parent != nullptr, n_cu, a.levels, a.slices);
      launch_accept_cluster(a, plan, a.patience >= 0 ? a.patience : 4000, ws + lay.msg_off, stream);
      return;
    }
  }
  SegStat* stats = reinterpret_cast<SegStat*>(ws);
  if (chain_path(a)) {
    AcceptParams P = accept_params(a, n_t_rows, c, stats);
    P.patience = (a.patience >= 0 && a.patience <= 1000000) ? a.patience : 1000;
    auto* msg = reinterpret_cast<unsigned long long*>(ws + chain_offset(a));
    unsigned long long* sums = msg + static_cast<size_t>(n_t_rows) * P.nseg * kChainWords;
    const MessageTag t = next_message_tag(false, stream);
    if (t.clear) clear_messages(msg, static_cast<int64_t>(chain_words(a)), stream);
    const int levels = a.max_nodes + 1;
    const dim3 grid(static_cast<unsigned>(static_cast<int64_t>(a.B) * levels * P.nseg));
    auto kernel = a.t_dtype == kBF16 ? (a.q_dtype == kBF16 ? chain_kernel<kBF16, kBF16>(a) : chain_kernel<kBF16, kF32>(a))
                                     : (a.q_dtype == kBF16 ? chain_kernel<kF32, kBF16>(a) : chain_kernel<kF32, kF32>(a));
    hipLaunchKernelGGL(kernel, grid, dim3(kLinThreads), 0, stream, P, msg, sums, t.tag, levels);
    return;
  }
  unsigned* words = reinterpret_cast<unsigned*>(ws + lay.words_off);      // start of the zeroed region
  // rows nobody was drawn from exist only when there are more draft rows than nodes
  const bool sparse_q = n_q_stat_rows > a.total_nodes;
  if (progressive_stats(a)) {
    unsigned* node_cnt = reinterpret_cast<unsigned*>(ws + lay.prog_cnt_off);
    int* stop = reinterpret_cast<int*>(ws + lay.prog_stop_off);
    unsigned* arrived0 = reinterpret_cast<unsigned*>(ws + lay.arrived_off);
    const int n_cnt = a.total_nodes;
    hipLaunchKernelGGL(accept_prog_init_kernel, dim3((n_cnt + kStatThreads - 1) / kStatThreads), dim3(kStatThreads), 0, stream,
                       node_cnt, n_cnt, stop, arrived0, a.B);
    const int nseg = stats_segments(a.V);
    const dim3 grid_p(nseg, a.B, 2 * a.max_nodes + 1);
    hipLaunchKernelGGL(row_stats_prog_kernel, grid_p, dim3(kStatThreads), 0, stream, a.target, a.t_dtype, n_t_rows,
                       a.draft_q, a.q_dtype, a.n_q_rows, a.V, c, nseg, stats, a.node_offsets, a.q_row, a.draft_tokens,
                       a.u_accept, node_cnt, stop, a.max_nodes);
  } else if (!a.target_stats_ready) {
    launch_row_stats(a.target, a.t_dtype, n_t_rows, a.draft_q, a.q_dtype, n_q_stat_rows, a.V, c, stats, stream, words,
                     static_cast<int>(lay.n_zero_words), sparse_q ? a.q_row : nullptr, a.total_nodes);
  } else if (n_q_stat_rows > 0) {
    // the target rows' entries were written by the LM-head kernel; only the draft rows are left
    launch_row_stats(nullptr, 0, 0, a.draft_q, a.q_dtype, n_q_stat_rows, a.V, c,
                     stats + static_cast<size_t>(n_t_rows) * stats_segments(a.V), stream, words,
                     static_cast<int>(lay.n_zero_words), sparse_q ? a.q_row : nullptr, a.total_nodes);
  } else {
    hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(kStatThreads), 0, stream, words,
                       static_cast<int>(lay.n_zero_words));
  }
  AcceptParams P = accept_params(a, n_t_rows, c, stats);
  P.desc = reinterpret_cast<PassDesc*>(ws + lay.desc_off);
  P.part = reinterpret_cast<PartSlot*>(ws + lay.part_off);
  if (linear_path(a)) {
    const int unit_classes = linear_unit_classes(a.B, a.V, n_cu);
    const int U = (a.V + unit_classes - 1) / unit_classes;
    P.parent = nullptr;
    double* partial = reinterpret_cast<double*>(ws + lay.lin_off);
    unsigned* arrived = reinterpret_cast<unsigned*>(ws + lay.arrived_off);
    const dim3 grid_l(static_cast<unsigned>(a.B) * U);
    const int blocks = unit_classes / kLinBlock;
    auto kernel = a.t_dtype == kBF16
                      ? (a.q_dtype == kBF16 ? linear_kernel<kBF16, kBF16>(blocks) : linear_kernel<kBF16, kF32>(blocks))
                      : (a.q_dtype == kBF16 ? linear_kernel<kF32, kBF16>(blocks) : linear_kernel<kF32, kF32>(blocks));
    hipLaunchKernelGGL(kernel, grid_l, dim3(kLinThreads), 0, stream, P, partial, arrived, U);
    return;
  }
  // Helpers pay when a pass is long against a hand-off between compute units (a few microseconds):
  // vocabularies of 64k classes and more; masters plus helpers stay within one workgroup per compute unit.
  int helpers = 0;
  if (a.V >= 65536) {
    helpers = n_cu / a.B - 1;
    helpers = helpers < 0 ? 0 : (helpers > kMaxHelpers ? kMaxHelpers : helpers);
  }
  if (a.helpers >= 0 && a.helpers <= kMaxHelpers && a.B * (1 + a.helpers) <= n_cu) helpers = a.helpers;   // per-call tuning
  P.helpers = helpers;
  P.patience = (a.patience >= 0 && a.patience <= 1000000) ? a.patience : 400;   // default: a few hundred microseconds
  const dim3 grid(a.B * (1 + helpers));
  const bool vec = (a.V % 8 == 0) && aligned16(a.target) && aligned16(a.draft_q);
  const bool fast = vec && a.V >= 8 && a.t_dtype == kBF16 && a.q_dtype == kBF16 && a.q_kind == 0;
  if (fast) hipLaunchKernelGGL(accept_walk_kernel<true>, grid, dim3(kWalkThreads), 0, stream, P);
  else hipLaunchKernelGGL(accept_walk_kernel<false>, grid, dim3(kWalkThreads), 0, stream, P);
}

}  // namespace specv
