// LM-head projection fused with the first pass of the vocab-wide softmax: the matrix product the
// paper singles out as the bulk of verification on the target model (Section 3.1), producing the
// logits o_i of Section 2.1 as bf16 together with the per-(row, 8192-class segment) statistics
// (maximum, sum of 2^((l - max) c)) that the acceptance walk starts from, so that the logits are
// never read back for that purpose and never exist in fp32.
//
//   logits[r, v] = bf16( sum_k hidden[r, k] * weight[v, k] ),  fp32 accumulation on the matrix cores.
//
// Vocabulary-as-M tiling: A = 32 weight rows, B = 32 hidden rows, so both operands of
// v_mfma_f32_32x32x16_bf16 are 16 contiguous bytes per lane of a row-major operand and no
// transpose is needed anywhere.  One workgroup = 8 waves = 4 vocabulary tiles x 2 halves of the
// contraction, producing a [128 vocab x 128 rows] block; the two halves are added through LDS.
// With up to 128 rows (a verification batch) the weight matrix is read exactly once and the kernel
// is bound by that read.  More rows go to a second kernel (below).
//
// Both operands are staged global -> registers -> LDS in 64-wide slices of the contraction
// (rows padded to 144 bytes: conflict-free 16-byte operand reads), the weights three slices ahead,
// one barrier per slice.  Weight slices are private to their wave; hidden slices are shared by the four waves of a
// half.
#include "common.h"
#include "kernels.h"

namespace specv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 lm_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float lm_f32x16;
typedef uint32_t lm_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t lm_u32x2 __attribute__((ext_vector_type(2)));

constexpr int kLmThreads = 512;
constexpr int kLmVB = 128;                          // vocabulary entries per workgroup (4 tiles of 32)
constexpr int kLmRB = 128;                          // hidden rows per workgroup (4 tiles of 32)
constexpr int kLmKC = 64;                           // contraction slice
constexpr int kLmPitch = kLmKC * 2 + 16;            // bytes per staged row
constexpr int kLmHidBuf = kLmRB * kLmPitch;         // one hidden slice
constexpr int kLmWBuf = 32 * kLmPitch;              // one weight slice of one wave
constexpr int kLmHidBytes = 2 * 2 * kLmHidBuf;      // 2 halves x 2 buffers
constexpr int kLmWBytes = 8 * 2 * kLmWBuf;          // 8 waves x 2 buffers
constexpr int kLmLds = kLmHidBytes + kLmWBytes;     // 147456 bytes
static_assert(4 * 64 * 64 * 4 <= kLmHidBytes, "split-K hand-over fits the hidden buffers");
static_assert(8192 / kLmVB <= kWave, "one wave merges one segment");

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

// Store the 32 vocabulary entries [vt, vt + 32) of one accumulator tile for this lane's row.  b[4 g + i] holds the
// lane's entry 8 g + 4 lh + i as bf16 bits.  full (uniform over the wave): the tile lies inside V, V is a multiple
// of 8 and the logits are 16-byte aligned; the two half-waves then exchange halves (lane ln ends up with all eight
// entries of group 2h, lane ln + 32 with those of group 2h + 1), so that every lane stores 16 bytes and one
// instruction writes 32 contiguous bytes per row - 8-byte stores left half of every 32-byte sector to a later
// instruction.
__device__ __forceinline__ void store_logit_tile(uint16_t* __restrict__ out_row, int vt, int lh, const uint32_t (&b)[16],
                                                 bool row_ok, bool full, int V) {
  if (full) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t w0x = b[8 * h + 0] | (b[8 * h + 1] << 16), w0y = b[8 * h + 2] | (b[8 * h + 3] << 16);
      const uint32_t w1x = b[8 * h + 4] | (b[8 * h + 5] << 16), w1y = b[8 * h + 6] | (b[8 * h + 7] << 16);
      const auto rx = __builtin_amdgcn_permlane32_swap(w0x, w1x, false, false);
      const auto ry = __builtin_amdgcn_permlane32_swap(w0y, w1y, false, false);
      lm_u32x4 v;
      v[0] = rx[0]; v[1] = ry[0]; v[2] = rx[1]; v[3] = ry[1];
      if (row_ok) *reinterpret_cast<lm_u32x4*>(out_row + vt + 8 * (2 * h + lh)) = v;
    }
  } else if (row_ok) {
    const bool vec4 = (V & 3) == 0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int vg = vt + 8 * g + 4 * lh;
      if (vec4 && vg + 3 < V) {
        lm_u32x2 w;
        w.x = b[4 * g] | (b[4 * g + 1] << 16);
        w.y = b[4 * g + 2] | (b[4 * g + 3] << 16);
        *reinterpret_cast<lm_u32x2*>(out_row + vg) = w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (vg + i < V) out_row[vg + i] = static_cast<uint16_t>(b[4 * g + i]);
      }
    }
  }
}

__global__ __launch_bounds__(kLmThreads) void lm_head_kernel(LmParams P) {
  extern __shared__ __align__(16) unsigned char lm_lds[];
  // consecutive logical blocks (the row blocks of one vocabulary block) on one XCD
  const int id = blockIdx.x;
  const int logical = (id & 7) * P.per_xcd + (id >> 3);
  if (logical >= P.total) return;
  const int rbk = logical % P.nrb, vb = logical / P.nrb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mt = wave & 3, kh = wave >> 2;
  const int ln = lane & 31, lh = lane >> 5;
  unsigned char* hid = lm_lds + kh * 2 * kLmHidBuf;
  unsigned char* wst = lm_lds + kLmHidBytes + wave * 2 * kLmWBuf;
  const int K2 = P.K >> 1;
  const int nch = K2 / kLmKC;
  const int kbase = kh * K2;
  const int v0 = vb * kLmVB + mt * 32;
  const int r0 = rbk * kLmRB;

  // staging: 8 lanes cover the 128 bytes of one row slice
  const int t = tid & 255;
  const uint16_t* wsrc[4];
  const uint16_t* hsrc[4];
  int wdst[4], hdst[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int vrow = v0 + (lane >> 3) + 8 * j;
    vrow = vrow < P.V ? vrow : P.V - 1;
    wsrc[j] = P.weight + static_cast<int64_t>(vrow) * P.K + kbase + (lane & 7) * 8;
    wdst[j] = ((lane >> 3) + 8 * j) * kLmPitch + (lane & 7) * 16;
    int hrow = r0 + (t >> 3) + 32 * j;
    hrow = hrow < P.rows ? hrow : P.rows - 1;
    hsrc[j] = P.hidden + static_cast<int64_t>(hrow) * P.K + kbase + (t & 7) * 8;
    hdst[j] = ((t >> 3) + 32 * j) * kLmPitch + (t & 7) * 16;
  }
  // Weight slices (HBM) are fetched three slices ahead into a ring of two register sets (slice s in
  // set (s - 1) % 2); hidden slices (L2) one slice ahead.  Loads past the end repeat the last slice
  // and are never used: a branch around a load would make the wait counts after it pessimistic.
  lm_u32x4 wring[2][4], hreg[4];
  auto load_w = [&](int c, lm_u32x4 (&w)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const lm_u32x4*>(wsrc[j] + c * kLmKC);
  };
  auto load_h = [&](int c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) hreg[j] = *reinterpret_cast<const lm_u32x4*>(hsrc[j] + c * kLmKC);
  };
  auto store_slice = [&](int buf, const lm_u32x4 (&w)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      *reinterpret_cast<lm_u32x4*>(wst + buf * kLmWBuf + wdst[j]) = w[j];
      *reinterpret_cast<lm_u32x4*>(hid + buf * kLmHidBuf + hdst[j]) = hreg[j];
    }
  };

  lm_f32x16 acc[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nt][r] = 0.f;

  const int last = nch - 1;
  load_w(0, wring[0]);
  load_h(0);
  store_slice(0, wring[0]);
  load_w(1 < last ? 1 : last, wring[0]);
  load_w(2 < last ? 2 : last, wring[1]);
  load_h(1 < last ? 1 : last);
  __syncthreads();
  for (int c0 = 0; c0 < nch; c0 += 2) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int c = c0 + r;
      if (c < nch) {
        const int buf = c & 1;
        const unsigned char* wrd = wst + buf * kLmWBuf + ln * kLmPitch + lh * 16;
        const unsigned char* hrd = hid + buf * kLmHidBuf + ln * kLmPitch + lh * 16;
#pragma unroll
        for (int s = 0; s < kLmKC / 16; ++s) {
          const lm_bf16x8 a = __builtin_bit_cast(lm_bf16x8, *reinterpret_cast<const lm_u32x4*>(wrd + 32 * s));
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) {
            const lm_bf16x8 b =
                __builtin_bit_cast(lm_bf16x8, *reinterpret_cast<const lm_u32x4*>(hrd + nt * 32 * kLmPitch + 32 * s));
            acc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[nt], 0, 0, 0);
          }
        }
        store_slice(buf ^ 1, wring[r]);                       // slice c + 1
        load_w(c + 3 < last ? c + 3 : last, wring[r]);
        load_h(c + 2 < last ? c + 2 : last);
        __syncthreads();
      }
    }
  }

  // add the two halves of the contraction: the upper half hands its tile over through LDS
  float* red = reinterpret_cast<float*>(lm_lds);
  if (kh == 1) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((mt * 64 + nt * 16 + r) << 6) + lane] = acc[nt][r];
  }
  __syncthreads();
  float2* sh_stat = reinterpret_cast<float2*>(lm_lds + kLmHidBytes);     // [4 tiles][128 rows]
  if (kh == 0) {
    const bool full = (P.V & 7) == 0 && v0 + 32 <= P.V && (reinterpret_cast<uintptr_t>(P.logits) & 15) == 0;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const int row = r0 + nt * 32 + ln;
      const bool row_ok = row < P.rows;
      uint16_t* out = P.logits + static_cast<int64_t>(row_ok ? row : 0) * P.V;
      float x[16];
      uint32_t b[16];
      float m = -INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int vg = v0 + 8 * g + 4 * lh;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * g + i;
          b[r] = f32_to_bf16_rne(acc[nt][r] + red[((mt * 64 + nt * 16 + r) << 6) + lane]);
          x[r] = (vg + i < P.V) ? __uint_as_float(b[r] << 16) : -INFINITY;
          m = fmaxf(m, x[r]);
        }
      }
      store_logit_tile(out, v0, lh, b, row_ok, full, P.V);
      const float mm = (m == -INFINITY) ? 0.f : m;
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) s += fast_exp2((x[r] - mm) * P.c);
      // the other half-wave holds the same row's other 16 classes
      const float mo = __shfl_xor(m, 32, kWave);
      const float so = __shfl_xor(s, 32, kWave);
      const float M = fmaxf(m, mo);
      const float MM = (M == -INFINITY) ? 0.f : M;
      const float mmo = (mo == -INFINITY) ? 0.f : mo;
      const float S = s * fast_exp2((mm - MM) * P.c) + so * fast_exp2((mmo - MM) * P.c);
      if (lh == 0) sh_stat[mt * kLmRB + nt * 32 + ln] = make_float2(M, S);
    }
  }
  __syncthreads();
  if (tid < kLmRB) {
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) M = fmaxf(M, sh_stat[i * kLmRB + tid].x);
    const float MM = (M == -INFINITY) ? 0.f : M;
    float S = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float2 st = sh_stat[i * kLmRB + tid];
      const float mi = (st.x == -INFINITY) ? 0.f : st.x;
      S += st.y * fast_exp2((mi - MM) * P.c);
    }
    const int row = r0 + tid;
    if (row < P.rows) P.bstats[static_cast<int64_t>(row) * P.nvb + vb] = make_float2(M, S);
  }
}

// ----------------------------------------------------------------------------------
// More than 128 rows.  A workgroup of 8 waves (two per SIMD, one workgroup per CU) computes [256 vocab x 16 NT2 rows];
// wave w owns 64 vocabulary entries, and the waves w and w + 4 (one SIMD) share the row tiles between them.  Both
// operands go from memory to LDS directly (global_load_lds, 16 bytes per lane, no registers) in 64-wide slices of the
// contraction, weights two slices ahead (they come from HBM).  The rows of a slice are 128 bytes without padding;
// 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7), so the 16 rows one operand read touches spread over all
// banks.
//
// Matrix work never waits for a barrier: the operands of a 32-deep step are read from LDS into registers while the
// step before is multiplied, across the slice boundary too.  The one barrier of a slice sits between its two steps:
// behind it every wave has read slice i completely (its buffers are refilled at once) and slice i + 1 has landed.
// ----------------------------------------------------------------------------------
constexpr int kTlThreads = 512;
constexpr int kTlVB = 256;                          // vocabulary entries per workgroup
constexpr int kTlSlice = 128;                       // bytes of a row per slice (64 bf16)
constexpr int kTlABuf = kTlVB * kTlSlice;           // one weight slice
constexpr int kTlABufs = 3;
constexpr int kTlOutPitch = kTlVB * 2 + 16;         // bytes per row of the output tile in LDS
// hidden slices: two ahead like the weights where the LDS (160 KB) allows, else one (they stay in L2)
constexpr int tl_bbufs(int NT2) { return NT2 <= 10 ? 3 : 2; }
constexpr int tl_lds(int NT2) {
  const int loop = kTlABufs * kTlABuf + tl_bbufs(NT2) * 16 * NT2 * kTlSlice;
  const int epi = 16 * NT2 * (kTlOutPitch + 4 * 8);          // output tile, then (max, sum) per row and vocabulary quarter
  return loop > epi ? loop : epi;
}
static_assert(tl_lds(16) <= 160 * 1024 && tl_lds(10) <= 160 * 1024, "one workgroup per compute unit");

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float lm_f32x4;

// 16 bytes per lane from base + off to LDS: lane i's land at byte lds_at + 16 i.  Not tracked by the compiler: the
// loop counts these loads itself (vmcnt).
__device__ __forceinline__ void load_to_lds(const unsigned char* base, unsigned off, unsigned lds_at) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_at), "v"(off), "s"(base) : "memory", "m0");
}

// The product of one wave with NT row tiles of the workgroup's NT2, up to the rounded output tile and the per-row
// statistics of its 64 vocabulary entries in LDS.  Waves of a workgroup may run it with different NT: every copy
// passes the same barriers and issues the same loads.
//
// What bounds it: the matrix cores under the chip's power limit (1024 x 4096 x 128256: busy 70 % of the cycles at
// 1.67 GHz).  A [64 vocab x 128 rows] tile per wave reads 12 KB of LDS per 32 matrix instructions (a third of the LDS
// rate) and a workgroup fetches 64 KB per 2048 matrix cycles; 16-row granularity keeps padded rows out of the products
// (1040 rows: 5 x 208).  Measured against the kernel this replaces (hidden operands packed by a kernel of their own and
// read from L2 by every wave, weights through registers): 1040 x 4096 x 128256 1095 -> 856 us (1.28 PFLOP/s), 429 x
// 8192 x 128256 909 -> 734 us, 512 x 4096 x 128256 506 -> 439 us, 224 x 4096 x 32000 89 -> 82 us, 200 x 8192 x 128256
// 563 -> 427 us (5.0 TB/s: bound by the weights from here down), 150 x 2048 x 8000 36 -> 19 us.
template <int NT2, int NT>
__device__ __forceinline__ void lm_tile_wave(const LmParams& P, unsigned char* lm_lds, int wave, int v0, int r0) {
  constexpr int kRows = 16 * NT2;
  constexpr int kBBufs = tl_bbufs(NT2);
  constexpr int kBBuf = kRows * kTlSlice;
  constexpr int kBLoads = kRows / 8;                // load instructions per hidden slice (8 rows each), dealt to 8 waves
  constexpr int kBPer = (kBLoads + 7) / 8;          // ... at most per wave
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int wm = wave & 3, row0 = (wave >> 2) * 16 * ((NT2 + 1) / 2);      // this wave's first row in the tile
  const int nch = P.K / 64, last = nch - 1;

  // ---- loads: instruction j of a wave covers 8 rows, 8 lanes per row ----
  const int lr = lane >> 3, lp = lane & 7;
  unsigned aoff[4], boff[kBPer];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ra = wave * 32 + j * 8 + lr;
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
    load_to_lds(abase + min(s, last) * kTlSlice, aoff[j], lds0 + buf * kTlABuf + (wave * 32 + j * 8) * kTlSlice);
  };
  auto load_b = [&](int s, int buf, int j) __attribute__((always_inline)) {
    if (8 * j + 7 < kBLoads || wave + 8 * j < kBLoads)
      load_to_lds(bbase + min(s, last) * kTlSlice, boff[j], lds0 + kTlABufs * kTlABuf + buf * kBBuf + (wave + 8 * j) * 8 * kTlSlice);
  };

  // ---- operand reads: lane l holds row l % 16 of a 16-row tile, contraction entries 8 (l / 16) .. + 8 of a 32-deep step ----
  const int pos0 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4;                  // step 0; step 1 is the same with bit 6 flipped
  const int a_lane = (wm * 64 + (lane & 15)) * kTlSlice + pos0;
  const int b_lane = kTlABufs * kTlABuf + (row0 + (lane & 15)) * kTlSlice + pos0;
  lm_u32x4 a0[4], b0[NT], a1[4], b1[NT];
  auto read_op = [&](int at, int t) { return *reinterpret_cast<const lm_u32x4*>(lm_lds + at + t * 16 * kTlSlice); };

  lm_f32x4 acc[4][NT];
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.f;

  // slices 0, 1, 2 of the weights and 0, 1 (2) of the hidden rows; then wait for slice 0
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    if (s < kBBufs)
#pragma unroll
      for (int j = 0; j < kBPer; ++j) load_b(s, s, j);
#pragma unroll
    for (int j = 0; j < 4; ++j) load_a(s, s, j);
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(8 + (kBBufs - 1) * (kBLoads / 8)) : "memory");
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int mi = 0; mi < 4; ++mi) a0[mi] = read_op(a_lane, mi);
#pragma unroll
  for (int ni = 0; ni < NT; ++ni) b0[ni] = read_op(b_lane, ni);

  // One 32-deep step: the products of (a, b) with the reads of the next step's operands (an, bn) between them.
  auto step = [&](const lm_u32x4 (&a)[4], const lm_u32x4 (&b)[NT], lm_u32x4 (&an)[4], lm_u32x4 (&bn)[NT], int a_at, int b_at,
                  auto&& extra) __attribute__((always_inline)) {
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) {
      // the 4 + NT operand reads spread over the first NT - 1 groups of four products
#pragma unroll
      for (int u = 0; u < 4 + NT; ++u)
        if (u * (NT - 1) / (4 + NT) == ni) {
          if (u < 4) an[u] = read_op(a_at, u);
          else bn[u - 4] = read_op(b_at, u - 4);
        }
      extra(ni);
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lm_bf16x8, a[mi]),
                                                              __builtin_bit_cast(lm_bf16x8, b[ni]), acc[mi][ni], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  int abuf = 0, bbuf = 0;                           // buffers of slice i
  for (int i = 0; i < nch; ++i) {
    const int anext = abuf == 2 ? 0 : abuf + 1;
    const int bnext = bbuf == kBBufs - 1 ? 0 : bbuf + 1;
    step(a0, b0, a1, b1, (a_lane + abuf * kTlABuf) ^ 64, (b_lane + bbuf * kBBuf) ^ 64, [](int) {});
    // this wave has read all of slice i (lgkmcnt) and its part of slice i + 1 is in LDS (vmcnt: the youngest loads,
    // of slice i + 2, may still be on their way)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(4 + (kBBufs - 2) * (kBLoads / 8)) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    step(a1, b1, a0, b0, a_lane + anext * kTlABuf, b_lane + bnext * kBBuf, [&](int ni) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 4 + kBPer; ++j)
        if (j * NT / (4 + kBPer) == ni) {
          if (j < kBPer) load_b(i + kBBufs, bbuf, j);
          else load_a(i + 3, abuf, j - kBPer);
        }
    });
    abuf = anext;
    bbuf = bnext;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();                      // the slice buffers are free

  // ---- round, statistics of the rounded values, output tile to LDS ----
  float2* sh_stat = reinterpret_cast<float2*>(lm_lds + kRows * kTlOutPitch);       // [4 vocabulary quarters][kRows]
  const int vg0 = wm * 64 + 4 * (lane >> 4);         // this lane's entries of tile mi: vg0 + 16 mi + 0..3
#pragma unroll
  for (int ni = 0; ni < NT; ++ni) {
    const int row = row0 + ni * 16 + (lane & 15);
    float x[4][4];
    float m = -INFINITY;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
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
      *reinterpret_cast<lm_u32x2*>(lm_lds + row * kTlOutPitch + (vg0 + 16 * mi) * 2) = w;
    }
    m = fmaxf(m, __shfl_xor(m, 16, kWave));
    m = fmaxf(m, __shfl_xor(m, 32, kWave));
    const float mm = (m == -INFINITY) ? 0.f : m;
    float s = 0.f;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += fast_exp2((x[mi][r] - mm) * P.c);
    s += __shfl_xor(s, 16, kWave);
    s += __shfl_xor(s, 32, kWave);
    if (lane < 16) sh_stat[wm * kRows + row] = make_float2(m, s);
  }
}

template <int NT2>
__global__ __launch_bounds__(kTlThreads) void lm_head_tile_kernel(LmParams P) {
  extern __shared__ __align__(16) unsigned char lm_lds[];
  constexpr int kRows = 16 * NT2;
  // the row blocks of one vocabulary block run next to each other on one XCD: its L2 serves the weights to all of them
  const int id = blockIdx.x;
  const int logical = (id & 7) * P.per_xcd + (id >> 3);
  if (logical >= P.total) return;
  const int rbk = logical % P.nrb, vb = logical / P.nrb;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int v0 = vb * kTlVB, r0 = rbk * kRows;
  if constexpr (NT2 % 2 == 0) {
    lm_tile_wave<NT2, NT2 / 2>(P, lm_lds, wave, v0, r0);
  } else {
    if (wave < 4) lm_tile_wave<NT2, (NT2 + 1) / 2>(P, lm_lds, wave, v0, r0);
    else lm_tile_wave<NT2, NT2 / 2>(P, lm_lds, wave, v0, r0);
  }
  __syncthreads();
  const float2* sh_stat = reinterpret_cast<const float2*>(lm_lds + kRows * kTlOutPitch);
  const int rows_here = min(kRows, P.rows - r0), cols = min(kTlVB, P.V - v0);
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
  if (cols == kTlVB && (P.V & 7) == 0 && (reinterpret_cast<uintptr_t>(P.logits) & 15) == 0) {
    for (int row = tid >> 5; row < rows_here; row += kTlThreads / 32)
      *reinterpret_cast<lm_u32x4*>(out + static_cast<int64_t>(row) * P.V + (tid & 31) * 8) =
          *reinterpret_cast<const lm_u32x4*>(lm_lds + row * kTlOutPitch + (tid & 31) * 16);
  } else {
    for (int i = tid; i < rows_here * kTlVB; i += kTlThreads) {
      const int row = i / kTlVB, v = i % kTlVB;
      if (v < cols) out[static_cast<int64_t>(row) * P.V + v] = *reinterpret_cast<const uint16_t*>(lm_lds + row * kTlOutPitch + v * 2);
    }
  }
}

template <int NT2>
static int launch_lm_tile(const LmParams& P, hipStream_t stream) {
  static std::atomic<uint64_t> attr_done{0};
  if (set_lds_once(&lm_head_tile_kernel<NT2>, tl_lds(NT2), attr_done) != 0) return -1;
  hipLaunchKernelGGL((lm_head_tile_kernel<NT2>), dim3(P.per_xcd * 8), dim3(kTlThreads), tl_lds(NT2), stream, P);
  return 0;
}

// Row tiles per workgroup: the split of the rows whose rounds over the chip cost least.  A slice costs its matrix work,
// proportional to the row tiles, plus a part that does not depend on them (weight traffic, barrier), about three tiles'
// worth.  Measured over all choices (us): 1040 x 4096 x 128256 13 tiles 856, 14 896, 12 943, 16 988, 10 972; 429 x 8192 x
// 128256 14 tiles 736, 15 771, 16 810, 10 831, 13 984; 224 x 4096 x 32000 8 tiles 81, 10 89, 14 92, 2 171; 150 x 2048 x
// 8000 2 tiles 19, 4 22, 14 42: the rule takes the fastest each time.
constexpr int kTlFixed = 3;
static int lm_tile_rows(int rows, int V, int n_cu) {
  static constexpr int kChoices[] = {16, 15, 14, 13, 12, 11, 10, 8, 6, 4, 2};
  const int64_t nvb = (V + kTlVB - 1) / kTlVB;
  int best = 16;
  int64_t best_cost = -1;
  for (const int nt2 : kChoices) {
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

// Workspace: block statistics, rows x ceil(V / 128) x 8 bytes (the kernel for more rows uses half of it).  The size that
// callers are told for more than 128 rows also covers a copy of the hidden states, which nothing uses at present: the
// answer of the size query stays what it was.
static size_t lm_bstats_bytes(int rows, int V) {
  const size_t nvb = (static_cast<size_t>(V) + kLmVB - 1) / kLmVB;
  return (static_cast<size_t>(rows) * nvb * sizeof(float2) + 255) / 256 * 256;
}

size_t lm_head_workspace_bytes(int rows, int d_model, int V) {
  size_t n = lm_bstats_bytes(rows, V) + 256;
  if (rows > kLmRB) n += static_cast<size_t>((rows + 31) / 32) * 32 * d_model * sizeof(uint16_t);
  return n;
}

size_t row_stats_bytes(int rows, int V) { return static_cast<size_t>(rows) * stats_segments(V) * sizeof(SegStat); }

int launch_lm_head(const LmHeadArgs& a, hipStream_t stream) {
  if (a.rows <= 0) return 0;
  LmParams P;
  P.rows = a.rows; P.K = a.d_model; P.V = a.V;
  P.c = kLog2e / a.temperature;
  P.hidden = static_cast<const uint16_t*>(a.hidden);
  P.weight = static_cast<const uint16_t*>(a.weight);
  P.logits = static_cast<uint16_t*>(a.logits);
  P.bstats = static_cast<float2*>(a.workspace);
  const bool tile = a.rows > kLmRB;
  const int vb = tile ? kTlVB : kLmVB;
  const int nt2 = tile ? lm_tile_rows(a.rows, a.V, current_device_cus()) : 0;
  const int rb = tile ? 16 * nt2 : kLmRB;
  P.nvb = (a.V + vb - 1) / vb;
  P.nrb = (a.rows + rb - 1) / rb;
  P.total = P.nvb * P.nrb;
  P.per_xcd = (P.total + 7) / 8;
  int rc = 0;
  switch (nt2) {
    case 0: {
      static std::atomic<uint64_t> attr_done{0};
      if (set_lds_once(&lm_head_kernel, kLmLds, attr_done) != 0) return -1;
      hipLaunchKernelGGL(lm_head_kernel, dim3(P.per_xcd * 8), dim3(kLmThreads), kLmLds, stream, P);
      break;
    }
    case 2: rc = launch_lm_tile<2>(P, stream); break;
    case 4: rc = launch_lm_tile<4>(P, stream); break;
    case 6: rc = launch_lm_tile<6>(P, stream); break;
    case 8: rc = launch_lm_tile<8>(P, stream); break;
    case 10: rc = launch_lm_tile<10>(P, stream); break;
    case 11: rc = launch_lm_tile<11>(P, stream); break;
    case 12: rc = launch_lm_tile<12>(P, stream); break;
    case 13: rc = launch_lm_tile<13>(P, stream); break;
    case 14: rc = launch_lm_tile<14>(P, stream); break;
    case 15: rc = launch_lm_tile<15>(P, stream); break;
    default: rc = launch_lm_tile<16>(P, stream); break;
  }
  if (rc != 0) return rc;
  const int nseg = stats_segments(a.V);
  hipLaunchKernelGGL(lm_stats_merge_kernel, dim3(nseg, a.rows), dim3(kWave), 0, stream, P.bstats, P.nvb, 8192 / vb, nseg, P.c,
                     static_cast<SegStat*>(a.stats));
  return 0;
}

}  // namespace specv
