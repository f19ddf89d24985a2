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

struct LmParams {
  int rows, K, V;
  int nvb, nrb, total, per_xcd;
  int slots;               // workgroups of an XCD
  float c;
  const uint16_t* hidden;
  const uint16_t* weight;
  uint16_t* logits;
  float2* bstats;          // [rows][nvb]
};

// Two fp32 values to bf16, round to nearest even: the first in the lower half.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
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
  static constexpr int kLoop = kABufs * kABuf + kBBufs * kBBuf;
  static constexpr int kStat = kRows * 4 * 8;                 // (max, sum) per row and vocabulary quarter
  // A workgroup takes several tiles one after the other, and its loads run on into the next, where the statistics have
  // room beside the slices.  Not with few rows: reading the weights alone evens out better over workgroups that start as
  // others end (8 x 4096 x 128256 174 us, 180 with fixed shares).
  static constexpr bool kStream = MI > 2 && kLoop + kStat <= kTlLds;
  static constexpr int kLds = kStream ? kLoop + kStat : (kLoop > kStat ? kLoop : kStat);
  static_assert(kLds <= kTlLds && kABufs >= 3 && kBBufs >= 2 && kABufs >= kBBufs, "one workgroup per compute unit");
};

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float lm_f32x4;

__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// op over the four lanes that are 16 and 32 apart: the same bits in all of them.
template <typename Op>
__device__ __forceinline__ float across16_32(float x, Op op) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned y = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto q = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return op(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// 16 bytes per lane from base + off to LDS: lane i's land at byte lds_at + 16 i.  Not tracked by the compiler: the
// loop counts these loads itself (vmcnt).  The LDS address is an operand bound to M0: the compiler writes that register
// itself and knows when it changes (a write inside the statement would have to be declared as a clobber, which it does
// not honour for a reserved register).
__device__ __forceinline__ void load_to_lds(const unsigned char* base, unsigned off, unsigned lds_at) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "{m0}"(lds_at), "v"(off), "s"(base) : "memory");
}

// The products of one wave with NT row tiles of the workgroup's NT2, for the workgroup's tiles first, first + slots, ...
// below end.  Waves of a workgroup may run it with different NT: every copy passes the same barriers and issues the same
// loads.
//
// What bounds it: with many rows the matrix cores under the chip's power limit (busy 70 % of the cycles at 1.8 GHz).  Of
// the 862 us of 1040 x 4096 x 128256 a fifth went into what does not depend on the contraction (20 thousand cycles per tile:
// first slices, output tile through LDS), so a workgroup now keeps its compute unit, the loads of its next tile go out
// under the last slices of the present one, and the logits go from the accumulators to memory (64 contiguous bytes per row
// and instruction after a swap between lanes) with no barrier but that of the statistics: 829 us (1.32 PFLOP/s), 429 x 8192
// x 128256 753 -> 733, 1040 x 1024 x 32000 73 -> 63, 512 x 4096 x 128256 437 -> 430.  With loads from memory left out the
// same loop takes 700, with the LDS reads left out too 630: what is left is mostly moving data.
// A [64 vocab x 128 rows] tile per wave reads 12 KB of LDS per 32 matrix instructions (a third of the LDS rate) and a
// workgroup fetches 64 KB per 2048 matrix cycles; 16-row granularity keeps padded rows out of the products (1040 rows: 5 x
// 208).
// With up to 128 rows the weights' way from HBM, with 128 vocabulary entries per workgroup and up to five slices ahead: 72
// x 4096 x 32000 45 us, 128 x 8192 x 128256 399, 8 x 4096 x 128256 173 = 6.1 TB/s, 30 x 8192 x 2000 30.
template <int MI, int NT2, int NT>
__device__ __forceinline__ void lm_tile_wave(const LmParams& P, unsigned char* lm_lds, int wave, int first, int end) {
  using C = TlCfg<MI, NT2>;
  constexpr int kRows = C::kRows, kVB = C::kVB;
  constexpr int kABufs = C::kABufs, kBBufs = C::kBBufs;
  constexpr int kABuf = C::kABuf, kBBuf = C::kBBuf;
  constexpr bool kStream = C::kStream;
  constexpr bool kOrdered = MI == 2 && NT2 == 2;
  constexpr int kBLoads = kRows / 8;                // load instructions per hidden slice (8 rows each), dealt to 8 waves
  constexpr int kBPer = (kBLoads + 7) / 8;          // ... at most per wave
  constexpr int kBMin = kBLoads / 8;                // ... at least
  constexpr int kStores = MI / 2 * NT;              // store instructions of a wave's logits
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int wm = wave & 3, row0 = (wave >> 2) * 16 * ((NT2 + 1) / 2);      // this wave's first row in the tile
  const int nch = P.K / 64;

  // ---- loads: instruction j of a wave covers 8 rows, 8 lanes per row.  Each operand has a cursor: the tile and slice
  // its next loads are of.  Behind the last tile it stays at the last slice (into a buffer nobody reads any more): every
  // slice issues the same loads ----
  // (opaque(lane): what is worked out from it once per tile is not kept in registers over the products)
  unsigned aoff[MI], boff[kBPer];
  const unsigned char *acur, *bcur;
  int atile, btile, aleft, bleft;
  auto seek_a = [&](int t) __attribute__((always_inline)) {
    const int v0 = __builtin_amdgcn_readfirstlane(t / P.nrb * kVB);
    acur = reinterpret_cast<const unsigned char*>(P.weight + static_cast<int64_t>(v0) * P.K);
    atile = t; aleft = nch;
    const int l = opaque(lane), lr = l >> 3, lp = l & 7;
#pragma unroll
    for (int j = 0; j < MI; ++j) {
      const int ra = (wave * MI + j) * 8 + lr;
      aoff[j] = static_cast<unsigned>(min(ra, P.V - 1 - v0)) * static_cast<unsigned>(P.K) * 2u + ((lp ^ ((ra >> 1) & 7)) << 4);
    }
  };
  auto seek_b = [&](int t) __attribute__((always_inline)) {
    const int r0 = __builtin_amdgcn_readfirstlane(t % P.nrb * kRows);
    bcur = reinterpret_cast<const unsigned char*>(P.hidden + static_cast<int64_t>(r0) * P.K);
    btile = t; bleft = nch;
    const int l = opaque(lane), lr = l >> 3, lp = l & 7;
#pragma unroll
    for (int j = 0; j < kBPer; ++j) {
      const int rb = (wave + 8 * j) * 8 + lr;
      boff[j] = static_cast<unsigned>(min(rb, P.rows - 1 - r0)) * static_cast<unsigned>(P.K) * 2u + ((lp ^ ((rb >> 1) & 7)) << 4);
    }
  };
  auto wrap_a = [&]() __attribute__((always_inline)) {
    if (atile + P.slots < end) seek_a(atile + P.slots);
    else { acur -= kTlSlice; aleft = 1; }
  };
  auto wrap_b = [&]() __attribute__((always_inline)) {
    if (btile + P.slots < end) seek_b(btile + P.slots);
    else { bcur -= kTlSlice; bleft = 1; }
  };
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) unsigned char*)lm_lds));
  auto load_a = [&](int buf, int j) __attribute__((always_inline)) {
    load_to_lds(acur, aoff[j], lds0 + buf * kABuf + (wave * MI + j) * 8 * kTlSlice);
  };
  auto load_b = [&](int buf, int j) __attribute__((always_inline)) {
    if (8 * j + 7 < kBLoads || wave + 8 * j < kBLoads)
      load_to_lds(bcur, boff[j], lds0 + kABufs * kABuf + buf * kBBuf + (wave + 8 * j) * 8 * kTlSlice);
  };

  // ---- operand reads: lane l holds row l % 16 of a 16-row tile, contraction entries 8 (l / 16) .. + 8 of a 32-deep step ----
  const int pos0 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4;                  // step 0; step 1 is the same with bit 6 flipped
  const int a_lane = (wm * 16 * MI + (lane & 15)) * kTlSlice + pos0;
  const int b_lane = kABufs * kABuf + (row0 + (lane & 15)) * kTlSlice + pos0;
  lm_u32x4 a0[MI], b0[NT], a1[MI], b1[NT];
  auto read_op = [&](int at, int t) { return *reinterpret_cast<const lm_u32x4*>(lm_lds + at + t * 16 * kTlSlice); };

  lm_f32x4 acc[MI][NT];
  int abuf = 0, bbuf = 0;                           // buffers of slice i

  // One 32-deep step: the products of (a, b) with the reads of the next step's operands (an, bn) between them.  The order
  // turns back at the end of a row of tiles, so that from one product to the next only one operand changes: less power
  // (429 x 8192 x 128256 746-773 -> 740-750 us; in registers alone 1985 -> 2015 TFLOP/s).
  // With one row tile in every wave (kOrdered) a step waits for memory, and its order is written down: a product, then the
  // reads.  Left to the compiler, weights from HBM / from the memory-side cache: 126 x 14336 x 3072 81.5 us instead of 80.2, 487 x
  // 12288 x 1216 63.6 / 43.6 instead of 62.4 / 43.4, 26 x 4096 x 3136 25.1 / 16.2 and 25.2 / 16.3.  Not with more row tiles, where
  // the like (loads, then products) is worth 3 % on 382 x 28672 x 4544 and costs 1 to 3 on 128 x 8192 x 16000 and 432 x 4096 x 2432.
  auto step = [&](const lm_u32x4 (&a)[MI], const lm_u32x4 (&b)[NT], lm_u32x4 (&an)[MI], lm_u32x4 (&bn)[NT], int a_at, int b_at,
                  auto&& extra) __attribute__((always_inline)) {
    constexpr int kAhead = kOrdered ? 1 : 0;
    auto product = [&](int mi, int ni) __attribute__((always_inline)) {
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lm_bf16x8, a[mi]),
                                                            __builtin_bit_cast(lm_bf16x8, b[ni]), acc[mi][ni], 0, 0, 0);
    };
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) {
      if constexpr (kAhead) {
        product(0, ni);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the MI + NT operand reads spread over the first NT - 1 groups of MI products
#pragma unroll
      for (int u = 0; u < MI + NT; ++u)
        if (u * (NT - 1) / (MI + NT) == ni) {
          if (u < MI) an[u] = read_op(a_at, u);
          else bn[u - MI] = read_op(b_at, u - MI);
        }
      extra(ni);
#pragma unroll
      for (int m = kAhead; m < MI; ++m) product(ni & 1 ? MI - 1 - m : m, ni);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  float2* sh_stat = reinterpret_cast<float2*>(lm_lds + (kStream ? C::kLoop : 0));       // [4 vocabulary quarters][kRows]
  bool stores_behind = false;      // kStores store instructions of this wave have gone out behind the loads of slices 0 and 1
  // the first slices, as many as there are buffers; then slice 0 is waited for and its first operands are read
  seek_a(first);
  seek_b(first);
  const unsigned char *const abase = acur, *const bbase = bcur;
  auto slice_of = [&](const unsigned char* base, int s) { return base + min(s, nch - 1) * kTlSlice; };
  auto first_loads = [&](int s) __attribute__((always_inline)) {
    if (s < kBBufs) {
#pragma unroll
      for (int j = 0; j < kBPer; ++j) load_b(s, j);
      if constexpr (kStream) {
        bcur += kTlSlice;
        if (--bleft == 0) wrap_b();
      } else {
        bcur += --bleft > 0 ? kTlSlice : 0;
      }
    }
#pragma unroll
    for (int j = 0; j < MI; ++j) load_a(s, j);
    if constexpr (kStream) {
      acur += kTlSlice;
      if (--aleft == 0) wrap_a();
    } else {
      acur += --aleft > 0 ? kTlSlice : 0;
    }
  };
  if constexpr (kStream) {
#pragma unroll 1
    for (int s = 0; s < kABufs; ++s) first_loads(s);
  } else {
#pragma unroll
    for (int s = 0; s < kABufs; ++s) first_loads(s);
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((kABufs - 1) * MI + (kBBufs - 1) * kBMin) : "memory");
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) a0[mi] = read_op(a_lane, mi);
#pragma unroll
  for (int ni = 0; ni < NT; ++ni) b0[ni] = read_op(b_lane, ni);

  for (int t = first;;) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NT; ++ni)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.f;

    // One slice i: its two steps, and the loads of slices i + kABufs and i + kBBufs (kOrdered: by the number, as there is one tile).
    auto slice = [&](int i, bool behind) __attribute__((always_inline)) {
      const int anext = abuf == kABufs - 1 ? 0 : abuf + 1;
      const int bnext = bbuf == kBBufs - 1 ? 0 : bbuf + 1;
      step(a0, b0, a1, b1, (a_lane + abuf * kABuf) ^ 64, (b_lane + bbuf * kBBuf) ^ 64, [](int) {});
      // this wave has read all of slice i (lgkmcnt) and its part of slice i + 1 is in LDS (vmcnt, which counts in order:
      // what was issued after the last of slice i + 1's two operands may still be on its way)
      constexpr int kAfterA = (kABufs - 2) * (kBMin + MI), kAfterB = (kBBufs - 2) * (kBMin + MI) + MI;
      constexpr int kAfter = kAfterA < kAfterB ? kAfterA : kAfterB;
      static_assert(kAfter + kStores < 64, "vmcnt has six bits");
      if (behind) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kAfter + kStores) : "memory");
      else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kAfter) : "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kOrdered) {
        acur = slice_of(abase, i + kABufs);
        bcur = slice_of(bbase, i + kBBufs);
      }
      step(a1, b1, a0, b0, a_lane + anext * kABuf, b_lane + bnext * kBBuf, [&](int ni) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MI + kBPer; ++j)
          if (j * NT / (MI + kBPer) == ni) {
            if (j < kBPer) load_b(bbuf, j);
            else load_a(abuf, j - kBPer);
          }
      });
      if constexpr (kStream) {
        acur += kTlSlice;
        bcur += kTlSlice;
      } else if constexpr (!kOrdered) {
        acur += --aleft > 0 ? kTlSlice : 0;
        bcur += --bleft > 0 ? kTlSlice : 0;
      }
      abuf = anext;
      bbuf = bnext;
    };
    if constexpr (kStream) {
      // in runs without the end of a tile for either cursor: a branch more per slice costs a tenth of the smallest ones
      for (int left = nch; left > 0;) {
        int run = min(left, min(aleft, bleft));
        left -= run; aleft -= run; bleft -= run;
        if (stores_behind) {
          slice(0, true);
          stores_behind = false;
          --run;
        }
        for (; run > 0; --run) slice(0, false);
        if (aleft == 0) wrap_a();
        if (bleft == 0) wrap_b();
      }
    } else if constexpr (kOrdered) {
      for (int i = 0; i < nch; ++i) slice(i, false);
    } else {
      for (int left = nch; left > 0; --left) slice(0, false);
    }
    if constexpr (!kStream) {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();                  // the slice buffers are free
    }

    // ---- round, statistics of the rounded values, logits.  A lane holds 4 entries of a row per tile; lanes 16 apart swap
    // them between tiles 2 p and 2 p + 1, and each has 8 ----
    const int v0 = __builtin_amdgcn_readfirstlane(t / P.nrb * kVB), r0 = __builtin_amdgcn_readfirstlane(t % P.nrb * kRows);
    const bool edge = v0 + kVB > P.V;
    unsigned char* out = reinterpret_cast<unsigned char*>(P.logits + static_cast<int64_t>(r0) * P.V + v0);
    const int el = opaque(lane), col = el & 15, g = el >> 4, vq = wm * 16 * MI, vst = vq + 16 * (g & 1) + 8 * (g >> 1);
#pragma unroll
    for (int ni = 0; ni < NT; ++ni) {
      const int row = row0 + ni * 16 + col;
      uint32_t w[MI][2];
      float x[MI][4];
      float m = -INFINITY;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          w[mi][h] = pack_bf16(acc[mi][ni][2 * h], acc[mi][ni][2 * h + 1]);
          x[mi][2 * h] = bf16_lo(w[mi][h]);
          x[mi][2 * h + 1] = bf16_hi(w[mi][h]);
        }
        if (edge)
#pragma unroll
          for (int r = 0; r < 4; ++r) x[mi][r] = v0 + vq + 16 * mi + 4 * g + r < P.V ? x[mi][r] : -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, x[mi][r]);
      }
      m = across16_32(m, [](float a, float b) { return fmaxf(a, b); });
      const float mm = (m == -INFINITY) ? 0.f : m;
      float s = 0.f;
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int r = 0; r < 4; ++r) s += fast_exp2((x[mi][r] - mm) * P.c);
      s = across16_32(s, [](float a, float b) { return a + b; });
      if (el < 16) sh_stat[wm * kRows + row] = make_float2(m, s);
      // rows past the last repeat it (their operands did): every wave issues every store
      const unsigned at = static_cast<unsigned>(min(row, P.rows - 1 - r0)) * static_cast<unsigned>(P.V) * 2u;
#pragma unroll
      for (int p = 0; p < MI / 2; ++p) {
        const auto lo = __builtin_amdgcn_permlane16_swap(w[2 * p][0], w[2 * p + 1][0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(w[2 * p][1], w[2 * p + 1][1], false, false);
        const raw4 q = {lo[0], hi[0], lo[1], hi[1]};
        const int v = vst + 32 * p;
        if (!edge || v0 + v + 8 <= P.V) {
          *reinterpret_cast<raw4_bf16*>(out + at + v * 2) = q;
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r)
            if (v0 + v + r < P.V) *reinterpret_cast<uint16_t*>(out + at + (v + r) * 2) = static_cast<uint16_t>(q[r / 2] >> (16 * (r & 1)));
        }
      }
    }
    stores_behind = kStream && !edge;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    const int row = wave * 64 + el;
    if (row < min(kRows, P.rows - r0)) {
      float M = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) M = fmaxf(M, sh_stat[i * kRows + row].x);
      const float MM = (M == -INFINITY) ? 0.f : M;
      float S = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 st = sh_stat[i * kRows + row];
        S += st.y * fast_exp2(((st.x == -INFINITY ? 0.f : st.x) - MM) * P.c);
      }
      P.bstats[static_cast<int64_t>(r0 + row) * P.nvb + t / P.nrb] = make_float2(M, S);
    }
    if constexpr (!kStream) break;
    t += P.slots;
    if (t >= end) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing is on its way to this workgroup's LDS when it ends
}

template <int MI, int NT2>
__global__ __launch_bounds__(kTlThreads) void lm_head_tile_kernel(LmParams P) {
  extern __shared__ __align__(16) unsigned char lm_lds[];
  // A workgroup takes every slots-th tile of its XCD's share.  The row blocks of one vocabulary block run next to each
  // other on one XCD: its L2 serves the weights to all of them.
  const int id = blockIdx.x;
  const int first = (id & 7) * P.per_xcd + (id >> 3), end = min(((id & 7) + 1) * P.per_xcd, P.total);
  if (first >= end) return;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  if constexpr (NT2 % 2 == 0) {
    lm_tile_wave<MI, NT2, NT2 / 2>(P, lm_lds, wave, first, end);
  } else {
    if (wave < 4) lm_tile_wave<MI, NT2, (NT2 + 1) / 2>(P, lm_lds, wave, first, end);
    else lm_tile_wave<MI, NT2, NT2 / 2>(P, lm_lds, wave, first, end);
  }
}

template <int MI, int NT2>
static int launch_lm_tile(LmParams P, hipStream_t stream) {
  static std::atomic<uint64_t> attr_done{0};
  constexpr int kLds = TlCfg<MI, NT2>::kLds;
  if (set_lds_once(&lm_head_tile_kernel<MI, NT2>, kLds, attr_done) != 0) return -1;
  if (!TlCfg<MI, NT2>::kStream) P.slots = P.per_xcd;
  hipLaunchKernelGGL((lm_head_tile_kernel<MI, NT2>), dim3(P.slots * 8), dim3(kTlThreads), kLds, stream, P);
  return 0;
}

// Row tiles per workgroup: the split of the rows whose rounds over the chip cost least.  A slice costs its matrix work,
// proportional to the row tiles, plus a part that does not depend on them (weight traffic, barrier), about three tiles'
// worth.  Measured over all choices (15 and 16 tiles leave no LDS to run on into the next tile), times as multiples of the
// fastest: 1040 x 4096 x 128256 13 tiles 1, 14 1.06, 11 1.06, 12 1.11, 16 1.19; 429 x 8192 x 128256 14 tiles 1, 15 1.06, 16 1.11, 10
// 1.15, 13 1.35; 224 x 4096 x 32000 8 tiles 1, 10 1.06, 13 1.11, 14 1.18; 700 x 4096 x 64000 15 tiles 1, 11 1.01, 16 1.05, 13 1.12;
// 256 x 4096 x 128256 16 tiles 1, 8 1.16; 200 x 8192 x 128256 13, 900 x 2048 x 100352 12, 300 x 4096 x 50304, 520 x 4096 x
// 32000 and 320 x 8192 x 32000 10: the rule takes the fastest of all ten.
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

// One wave per (row, 8192-class segment), four to a workgroup: the block statistics of the segment (per_seg <= 64 of them)
// become the entry the acceptance walk reads.  (One wave per workgroup, a launch of thousands: 72 rows x 4 segments 4.7 -> 4.4 us,
// 429 x 16 5.5 -> 5.2, 1040 x 16 7.0 -> 6.2.)
constexpr int kMergeWaves = 4;
__global__ __launch_bounds__(kMergeWaves * kWave) void lm_stats_merge_kernel(const float2* __restrict__ bstats, int nvb, int per_seg, int nseg,
                                                                             int entries, float c, SegStat* __restrict__ stats) {
  const int entry = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * kMergeWaves + threadIdx.x / kWave)), lane = threadIdx.x & 63;
  if (entry >= entries) return;
  const int row = entry / nseg, seg = entry - row * nseg;
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
    stats[entry] = st;
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
  P.slots = std::max(1, std::min(P.per_xcd, current_device_cus() / 8));
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
  hipLaunchKernelGGL(lm_stats_merge_kernel, dim3((a.rows * nseg + kMergeWaves - 1) / kMergeWaves), dim3(kMergeWaves * kWave), 0, stream, P.bstats, P.nvb,
                     8192 / vb, nseg, a.rows * nseg, P.c,
                     static_cast<SegStat*>(a.stats));
  return 0;
}

}  // namespace specv
