// LM-head projection fused with the first pass of the vocab-wide softmax: the matrix product the
// paper singles out as the bulk of verification on the target model (Section 3.1), producing the
// logits o_i of Section 2.1 as bf16 together with the per-(row, 8192-class segment) statistics
// (maximum, sum of 2^((l - max) c)) that the acceptance walk starts from, so that the logits are
// never read back for that purpose and never exist in fp32.
//
//   logits[r, v] = bf16( sum_k hidden[r, k] * weight[v, k] ),  fp32 accumulation on the matrix cores.
//
// Vocabulary-as-M tiling: A = 16 weight rows, B = 16 hidden rows, so both operands of v_mfma_f32_16x16x32_bf16 are 16
// contiguous bytes per lane of a row-major operand and no transpose is needed anywhere.  Up to a few hundred rows the
// kernel is bound by reading the weight matrix once, beyond by the matrix cores.
#include "common.h"
#include "kernels.h"

namespace specv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 lm_bf16x8;
typedef uint32_t lm_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t lm_u32x2 __attribute__((ext_vector_type(2)));

struct LmParams {
  int rows, K, V;
  int nvb, nrb, total, per_xcd;
  float c;
  const uint16_t* hidden;
  const uint16_t* weight;
  uint16_t* logits;
  float2* bstats;          // [rows][nvb]
};

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

// ----------------------------------------------------------------------------------
// A workgroup of 8 waves (two per SIMD, one workgroup per CU) computes [64 MI vocab x 16 NT2 rows]; wave w owns 16 MI
// vocabulary entries, and the waves w and w + 4 (one SIMD) share the row tiles between them.  Both operands go from
// memory to LDS directly (global_load_lds, 16 bytes per lane, no registers) in 64-wide slices of the contraction,
// weights two slices ahead and more (they come from HBM).  The rows of a slice are 128 bytes without padding; 16-byte
// chunk c of row r sits at position c ^ ((r >> 1) & 7), so the 16 rows one operand read touches spread over all banks.
//
// Matrix work never waits for a barrier: the operands of a 32-deep step are read from LDS into registers while the
// step before is multiplied, across the slice boundary too.  The one barrier of a slice sits between its two steps:
// behind it every wave has read slice i completely (its buffers are refilled at once) and slice i + 1 has landed.
// ----------------------------------------------------------------------------------
constexpr int kTlThreads = 512;
constexpr int kTlSlice = 128;                       // bytes of a row per slice (64 bf16)
constexpr int kTlLds = 160 * 1024;
template <int MI, int NT2>
struct TlCfg {
  static constexpr int kVB = 64 * MI;                         // vocabulary entries per workgroup
  static constexpr int kRows = 16 * NT2;
  static constexpr int kABuf = kVB * kTlSlice, kBBuf = kRows * kTlSlice;
  // 128 vocabulary entries (few rows, bound by the weights): as many slices as fit, at most six.  256: three of the
  // weights, and of the hidden rows three or, where the LDS ends, two (they stay in L2).
  static constexpr int kFit = kTlLds / (kABuf + kBBuf) < 6 ? kTlLds / (kABuf + kBBuf) : 6;
  static constexpr int kABufs = MI == 2 ? kFit : 3;
  static constexpr int kBBufs = MI == 2 ? kFit : (NT2 <= 10 ? 3 : 2);
  static constexpr int kOutPitch = kVB * 2 + 16;              // bytes per row of the output tile in LDS
  static constexpr int kLoop = kABufs * kABuf + kBBufs * kBBuf;
  static constexpr int kEpi = kRows * (kOutPitch + 4 * 8);    // output tile, then (max, sum) per row and vocabulary quarter
  static constexpr int kLds = kLoop > kEpi ? kLoop : kEpi;
  static_assert(kLds <= kTlLds && kABufs >= 3 && kBBufs >= 2 && kABufs >= kBBufs, "one workgroup per compute unit");
};

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float lm_f32x4;

// 16 bytes per lane from base + off to LDS: lane i's land at byte lds_at + 16 i.  Not tracked by the compiler: the
// loop counts these loads itself (vmcnt).  The LDS address is an operand bound to M0: the compiler writes that register
// itself and knows when it changes (a write inside the statement would have to be declared as a clobber, which it does
// not honour for a reserved register).
__device__ __forceinline__ void load_to_lds(const unsigned char* base, unsigned off, unsigned lds_at) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "{m0}"(lds_at), "v"(off), "s"(base) : "memory");
}

// The product of one wave with NT row tiles of the workgroup's NT2, up to the rounded output tile and the per-row
// statistics of its 64 vocabulary entries in LDS.  Waves of a workgroup may run it with different NT: every copy
// passes the same barriers and issues the same loads.
//
// What bounds it: with many rows the matrix cores under the chip's power limit (1024 x 4096 x 128256: busy 70 % of the
// cycles at 1.67 GHz).  A [64 vocab x 128 rows] tile per wave reads 12 KB of LDS per 32 matrix instructions (a third of the
// LDS rate) and a workgroup fetches 64 KB per 2048 matrix cycles; 16-row granularity keeps padded rows out of the products
// (1040 rows: 5 x 208).  Measured in loops, against the kernel this replaces (hidden operands packed by a kernel of their
// own and read from L2 by every wave, weights through registers): 1040 x 4096 x 128256 1091 -> 870 us (1.26 PFLOP/s),
// 429 x 8192 x 128256 908 -> 758 us, 512 x 4096 x 128256 507 -> 437 us, 224 x 4096 x 32000 85 -> 75 us, 200 x 8192 x
// 128256 581 -> 458 us (4.7 TB/s).
// With up to 128 rows the weights' way from HBM, with 128 vocabulary entries per workgroup and up to five slices ahead
// (a kernel that staged them through registers, three slices ahead, in brackets): 72 x 4096 x 32000 61 us (68), 128 x
// 8192 x 128256 402 (449), 8 x 4096 x 128256 178 = 5.9 TB/s (202), 30 x 8192 x 2000 30 (71), 100 x 4096 x 8000 28 (48).
template <int MI, int NT2, int NT>
__device__ __forceinline__ void lm_tile_wave(const LmParams& P, unsigned char* lm_lds, int wave, int v0, int r0) {
  using C = TlCfg<MI, NT2>;
  constexpr int kRows = C::kRows;
  constexpr int kABufs = C::kABufs, kBBufs = C::kBBufs;
  constexpr int kABuf = C::kABuf, kBBuf = C::kBBuf;
  constexpr int kBLoads = kRows / 8;                // load instructions per hidden slice (8 rows each), dealt to 8 waves
  constexpr int kBPer = (kBLoads + 7) / 8;          // ... at most per wave
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int wm = wave & 3, row0 = (wave >> 2) * 16 * ((NT2 + 1) / 2);      // this wave's first row in the tile
  const int nch = P.K / 64, last = nch - 1;

  // ---- loads: instruction j of a wave covers 8 rows, 8 lanes per row ----
  const int lr = lane >> 3, lp = lane & 7;
  unsigned aoff[MI], boff[kBPer];
#pragma unroll
  for (int j = 0; j < MI; ++j) {
    const int ra = (wave * MI + j) * 8 + lr;
    aoff[j] = static_cast<unsigned>(min(ra, P.V - 1 - v0)) * static_cast<unsigned>(P.K) * 2u + ((lp ^ ((ra >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int j = 0; j < kBPer; ++j) {
    const int rb = (wave + 8 * j) * 8 + lr;
    boff[j] = static_cast<unsigned>(min(rb, P.rows - 1 - r0)) * static_cast<unsigned>(P.K) * 2u + ((lp ^ ((rb >> 1) & 7)) << 4);
  }
  const unsigned char* abase = reinterpret_cast<const unsigned char*>(P.weight + static_cast<int64_t>(v0) * P.K);
  const unsigned char* bbase = reinterpret_cast<const unsigned char*>(P.hidden + static_cast<int64_t>(r0) * P.K);
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) unsigned char*)lm_lds));
  // slices past the end repeat the last one into a buffer nobody reads any more: every slice issues the same loads
  auto load_a = [&](int s, int buf, int j) __attribute__((always_inline)) {
    load_to_lds(abase + min(s, last) * kTlSlice, aoff[j], lds0 + buf * kABuf + (wave * MI + j) * 8 * kTlSlice);
  };
  auto load_b = [&](int s, int buf, int j) __attribute__((always_inline)) {
    if (8 * j + 7 < kBLoads || wave + 8 * j < kBLoads)
      load_to_lds(bbase + min(s, last) * kTlSlice, boff[j], lds0 + kABufs * kABuf + buf * kBBuf + (wave + 8 * j) * 8 * kTlSlice);
  };

  // ---- operand reads: lane l holds row l % 16 of a 16-row tile, contraction entries 8 (l / 16) .. + 8 of a 32-deep step ----
  const int pos0 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4;                  // step 0; step 1 is the same with bit 6 flipped
  const int a_lane = (wm * 16 * MI + (lane & 15)) * kTlSlice + pos0;
  const int b_lane = kABufs * kABuf + (row0 + (lane & 15)) * kTlSlice + pos0;
  lm_u32x4 a0[MI], b0[NT], a1[MI], b1[NT];
  auto read_op = [&](int at, int t) { return *reinterpret_cast<const lm_u32x4*>(lm_lds + at + t * 16 * kTlSlice); };

  lm_f32x4 acc[MI][NT];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.f;

  // the first slices, as many as there are buffers; then wait for slice 0
#pragma unroll
  for (int s = 0; s < kABufs; ++s) {
    if (s < kBBufs)
#pragma unroll
      for (int j = 0; j < kBPer; ++j) load_b(s, s, j);
#pragma unroll
    for (int j = 0; j < MI; ++j) load_a(s, s, j);
  }
  constexpr int kBMin = kBLoads / 8;                // load_b instructions of a slice in every wave, at least
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kABufs - 1) * MI + (kBBufs - 1) * kBMin) : "memory");
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) a0[mi] = read_op(a_lane, mi);
#pragma unroll
  for (int ni = 0; ni < NT; ++ni) b0[ni] = read_op(b_lane, ni);

  // One 32-deep step: the products of (a, b) with the reads of the next step's operands (an, bn) between them.
  auto step = [&](const lm_u32x4 (&a)[MI], const lm_u32x4 (&b)[NT], lm_u32x4 (&an)[MI], lm_u32x4 (&bn)[NT], int a_at, int b_at,
                  auto&& extra) __attribute__((always_inline)) {
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) {
      // the MI + NT operand reads spread over the first NT - 1 groups of MI products
#pragma unroll
      for (int u = 0; u < MI + NT; ++u)
        if (u * (NT - 1) / (MI + NT) == ni) {
          if (u < MI) an[u] = read_op(a_at, u);
          else bn[u - MI] = read_op(b_at, u - MI);
        }
      extra(ni);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lm_bf16x8, a[mi]),
                                                              __builtin_bit_cast(lm_bf16x8, b[ni]), acc[mi][ni], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  int abuf = 0, bbuf = 0;                           // buffers of slice i
  for (int i = 0; i < nch; ++i) {
    const int anext = abuf == kABufs - 1 ? 0 : abuf + 1;
    const int bnext = bbuf == kBBufs - 1 ? 0 : bbuf + 1;
    step(a0, b0, a1, b1, (a_lane + abuf * kABuf) ^ 64, (b_lane + bbuf * kBBuf) ^ 64, [](int) {});
    // this wave has read all of slice i (lgkmcnt) and its part of slice i + 1 is in LDS (vmcnt: what was issued after
    // the last of slice i + 1's two operands may still be on its way)
    constexpr int kAfterA = (kABufs - 2) * (kBMin + MI), kAfterB = (kBBufs - 2) * (kBMin + MI) + MI;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kAfterA < kAfterB ? kAfterA : kAfterB) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    step(a1, b1, a0, b0, a_lane + anext * kABuf, b_lane + bnext * kBBuf, [&](int ni) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < MI + kBPer; ++j)
        if (j * NT / (MI + kBPer) == ni) {
          if (j < kBPer) load_b(i + kBBufs, bbuf, j);
          else load_a(i + kABufs, abuf, j - kBPer);
        }
    });
    abuf = anext;
    bbuf = bnext;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();                      // the slice buffers are free

  // ---- round, statistics of the rounded values, output tile to LDS ----
  float2* sh_stat = reinterpret_cast<float2*>(lm_lds + kRows * C::kOutPitch);       // [4 vocabulary quarters][kRows]
  const int vg0 = wm * 16 * MI + 4 * (lane >> 4);         // this lane's entries of tile mi: vg0 + 16 mi + 0..3
#pragma unroll
  for (int ni = 0; ni < NT; ++ni) {
    const int row = row0 + ni * 16 + (lane & 15);
    float x[MI][4];
    float m = -INFINITY;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      uint32_t b[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        b[r] = f32_to_bf16_rne(acc[mi][ni][r]);
        x[mi][r] = (v0 + vg0 + 16 * mi + r < P.V) ? __uint_as_float(b[r] << 16) : -INFINITY;
        m = fmaxf(m, x[mi][r]);
      }
      lm_u32x2 w;
      w.x = b[0] | (b[1] << 16);
      w.y = b[2] | (b[3] << 16);
      *reinterpret_cast<lm_u32x2*>(lm_lds + row * C::kOutPitch + (vg0 + 16 * mi) * 2) = w;
    }
    m = fmaxf(m, __shfl_xor(m, 16, kWave));
    m = fmaxf(m, __shfl_xor(m, 32, kWave));
    const float mm = (m == -INFINITY) ? 0.f : m;
    float s = 0.f;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += fast_exp2((x[mi][r] - mm) * P.c);
    s += __shfl_xor(s, 16, kWave);
    s += __shfl_xor(s, 32, kWave);
    if (lane < 16) sh_stat[wm * kRows + row] = make_float2(m, s);
  }
}

template <int MI, int NT2>
__global__ __launch_bounds__(kTlThreads) void lm_head_tile_kernel(LmParams P) {
  extern __shared__ __align__(16) unsigned char lm_lds[];
  using C = TlCfg<MI, NT2>;
  constexpr int kRows = C::kRows, kVB = C::kVB;
  // the row blocks of one vocabulary block run next to each other on one XCD: its L2 serves the weights to all of them
  const int id = blockIdx.x;
  const int logical = (id & 7) * P.per_xcd + (id >> 3);
  if (logical >= P.total) return;
  const int rbk = logical % P.nrb, vb = logical / P.nrb;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int v0 = vb * kVB, r0 = rbk * kRows;
  if constexpr (NT2 % 2 == 0) {
    lm_tile_wave<MI, NT2, NT2 / 2>(P, lm_lds, wave, v0, r0);
  } else {
    if (wave < 4) lm_tile_wave<MI, NT2, (NT2 + 1) / 2>(P, lm_lds, wave, v0, r0);
    else lm_tile_wave<MI, NT2, NT2 / 2>(P, lm_lds, wave, v0, r0);
  }
  __syncthreads();
  const float2* sh_stat = reinterpret_cast<const float2*>(lm_lds + kRows * C::kOutPitch);
  const int rows_here = min(kRows, P.rows - r0), cols = min(kVB, P.V - v0);
  if (tid < rows_here) {
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) M = fmaxf(M, sh_stat[i * kRows + tid].x);
    const float MM = (M == -INFINITY) ? 0.f : M;
    float S = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float2 st = sh_stat[i * kRows + tid];
      S += st.y * fast_exp2(((st.x == -INFINITY ? 0.f : st.x) - MM) * P.c);
    }
    P.bstats[static_cast<int64_t>(r0 + tid) * P.nvb + vb] = make_float2(M, S);
  }
  uint16_t* out = P.logits + static_cast<int64_t>(r0) * P.V + v0;
  constexpr int kLanes = kVB / 8;                    // lanes that write a row, 16 bytes each
  if (cols == kVB && (P.V & 7) == 0 && (reinterpret_cast<uintptr_t>(P.logits) & 15) == 0) {
    for (int row = tid / kLanes; row < rows_here; row += kTlThreads / kLanes)
      *reinterpret_cast<lm_u32x4*>(out + static_cast<int64_t>(row) * P.V + (tid % kLanes) * 8) =
          *reinterpret_cast<const lm_u32x4*>(lm_lds + row * C::kOutPitch + (tid % kLanes) * 16);
  } else {
    for (int i = tid; i < rows_here * kVB; i += kTlThreads) {
      const int row = i / kVB, v = i % kVB;
      if (v < cols) out[static_cast<int64_t>(row) * P.V + v] = *reinterpret_cast<const uint16_t*>(lm_lds + row * C::kOutPitch + v * 2);
    }
  }
}

template <int MI, int NT2>
static int launch_lm_tile(const LmParams& P, hipStream_t stream) {
  static std::atomic<uint64_t> attr_done{0};
  constexpr int kLds = TlCfg<MI, NT2>::kLds;
  if (set_lds_once(&lm_head_tile_kernel<MI, NT2>, kLds, attr_done) != 0) return -1;
  hipLaunchKernelGGL((lm_head_tile_kernel<MI, NT2>), dim3(P.per_xcd * 8), dim3(kTlThreads), kLds, stream, P);
  return 0;
}

// Row tiles per workgroup: the split of the rows whose rounds over the chip cost least.  A slice costs its matrix work,
// proportional to the row tiles, plus a part that does not depend on them (weight traffic, barrier), about three tiles'
// worth.  Measured over all choices, times as multiples of the fastest: 1040 x 4096 x 128256 13 tiles 1, 14 1.05, 12 1.10,
// 10 1.14, 16 1.15; 429 x 8192 x 128256 14 tiles 1, 15 1.05, 16 1.10, 10 1.13, 13 1.34; 224 x 4096 x 32000 8 tiles 1, 10
// 1.10, 14 1.14: the rule takes the fastest each time.
constexpr int kTlFixed = 3;
template <int N>
static int lm_tile_rows(const int (&choices)[N], int vb, int rows, int V, int n_cu) {
  const int64_t nvb = (V + vb - 1) / vb;
  int best = choices[0];
  int64_t best_cost = -1;
  for (const int nt2 : choices) {
    const int64_t nrb = (rows + 16 * nt2 - 1) / (16 * nt2);
    const int64_t cost = ((nvb * nrb + n_cu - 1) / n_cu) * (nt2 + kTlFixed);
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = nt2; }
  }
  return best;
}

// One wave per (row, 8192-class segment): the block statistics of the segment (per_seg <= 64 of them) become the
// entry the acceptance walk reads.
__global__ __launch_bounds__(kWave) void lm_stats_merge_kernel(const float2* __restrict__ bstats, int nvb, int per_seg, int nseg,
                                                               float c, SegStat* __restrict__ stats) {
  const int seg = blockIdx.x, row = blockIdx.y, lane = threadIdx.x;
  const int i = seg * per_seg + lane;
  float m = -INFINITY, s = 0.f;
  if (lane < per_seg && i < nvb) {
    const float2 b = bstats[static_cast<int64_t>(row) * nvb + i];
    m = b.x; s = b.y;
  }
  const float M = wave_max(m);
  const float MM = (M == -INFINITY) ? 0.f : M;
  const float mm = (m == -INFINITY) ? 0.f : m;
  const double z = wave_sum(static_cast<double>(s) * static_cast<double>(fast_exp2((mm - MM) * c)));
  if (lane == 0) {
    SegStat st;
    st.m = M; st.pad = 0.f; st.z = z;
    stats[static_cast<int64_t>(row) * nseg + seg] = st;
  }
}

// Workspace: block statistics, rows x ceil(V / 128) x 8 bytes (workgroups of 256 vocabulary entries use half of it).  The size that
// callers are told for more than 128 rows also covers a copy of the hidden states, which nothing uses at present: the
// answer of the size query stays what it was.
static size_t lm_bstats_bytes(int rows, int V) {
  const size_t nvb = (static_cast<size_t>(V) + 127) / 128;
  return (static_cast<size_t>(rows) * nvb * sizeof(float2) + 255) / 256 * 256;
}

size_t lm_head_workspace_bytes(int rows, int d_model, int V) {
  size_t n = lm_bstats_bytes(rows, V) + 256;
  if (rows > 128) n += static_cast<size_t>((rows + 31) / 32) * 32 * d_model * sizeof(uint16_t);
  return n;
}

size_t row_stats_bytes(int rows, int V) { return static_cast<size_t>(rows) * stats_segments(V) * sizeof(SegStat); }

LmHeadPlan make_lm_head_plan(int rows, int V) {
  static constexpr int kFew[] = {8, 6, 5, 4, 3, 2}, kMany[] = {16, 15, 14, 13, 12, 11, 10, 8, 6, 4};
  const int n_cu = current_device_cus();
  // 128 vocabulary entries per workgroup, more slices ahead: few rows (bound by the weights: twice the workgroups fetch
  // them), and products too small to give every compute unit a workgroup of 256 entries and two row tiles (300 x 16384 x
  // 4096 154 -> 96 us, 600 x 4096 x 3000 33 -> 23, 150 x 2048 x 8000 19 -> 14).
  const bool few = rows <= 128 || static_cast<int64_t>((V + 255) / 256) * ((rows + 31) / 32) <= n_cu;
  LmHeadPlan p;
  p.vocab_block = few ? 128 : 256;
  p.row_tiles = few ? lm_tile_rows(kFew, p.vocab_block, rows, V, n_cu) : lm_tile_rows(kMany, p.vocab_block, rows, V, n_cu);
  return p;
}

int launch_lm_head(const LmHeadArgs& a, hipStream_t stream) {
  if (a.rows <= 0) return 0;
  LmParams P;
  P.rows = a.rows; P.K = a.d_model; P.V = a.V;
  P.c = kLog2e / a.temperature;
  P.hidden = static_cast<const uint16_t*>(a.hidden);
  P.weight = static_cast<const uint16_t*>(a.weight);
  P.logits = static_cast<uint16_t*>(a.logits);
  P.bstats = static_cast<float2*>(a.workspace);
  const LmHeadPlan plan = make_lm_head_plan(a.rows, a.V);
  const int vb = plan.vocab_block, nt2 = plan.row_tiles;
  const int rb = 16 * nt2;
  P.nvb = (a.V + vb - 1) / vb;
  P.nrb = (a.rows + rb - 1) / rb;
  P.total = P.nvb * P.nrb;
  P.per_xcd = (P.total + 7) / 8;
  int rc = -1;
  switch (nt2 + (vb == 128 ? 100 : 0)) {
    case 102: rc = launch_lm_tile<2, 2>(P, stream); break;
    case 103: rc = launch_lm_tile<2, 3>(P, stream); break;
    case 104: rc = launch_lm_tile<2, 4>(P, stream); break;
    case 105: rc = launch_lm_tile<2, 5>(P, stream); break;
    case 106: rc = launch_lm_tile<2, 6>(P, stream); break;
    case 108: rc = launch_lm_tile<2, 8>(P, stream); break;
    case 4: rc = launch_lm_tile<4, 4>(P, stream); break;
    case 6: rc = launch_lm_tile<4, 6>(P, stream); break;
    case 8: rc = launch_lm_tile<4, 8>(P, stream); break;
    case 10: rc = launch_lm_tile<4, 10>(P, stream); break;
    case 11: rc = launch_lm_tile<4, 11>(P, stream); break;
    case 12: rc = launch_lm_tile<4, 12>(P, stream); break;
    case 13: rc = launch_lm_tile<4, 13>(P, stream); break;
    case 14: rc = launch_lm_tile<4, 14>(P, stream); break;
    case 15: rc = launch_lm_tile<4, 15>(P, stream); break;
    case 16: rc = launch_lm_tile<4, 16>(P, stream); break;
  }
  if (rc != 0) return rc;
  const int nseg = stats_segments(a.V);
  hipLaunchKernelGGL(lm_stats_merge_kernel, dim3(nseg, a.rows), dim3(kWave), 0, stream, P.bstats, P.nvb, 8192 / vb, nseg, P.c,
                     static_cast<SegStat*>(a.stats));
  return 0;
}

}  // namespace specv
