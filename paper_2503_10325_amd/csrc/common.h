// Device helpers shared by the gfx950 kernels of the verification library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace specv {

constexpr int kWave = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr double kLn2 = 0.6931471805599453;

// dtype codes of the C ABI (spec_dtype)
constexpr int kBF16 = 0;
constexpr int kF32 = 1;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// 2^x through the hardware transcendental unit.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// One logit of a row-major [rows, V] matrix of either dtype, as fp32 (exact for bf16).
__device__ __forceinline__ float load_logit(const void* base, int dtype, int64_t idx) {
  if (dtype == kBF16) return bf16_bits_to_float(static_cast<const uint16_t*>(base)[idx]);
  return static_cast<const float*>(base)[idx];
}

// Eight consecutive logits of one row starting at element e0; positions >= V read as -inf.  The 16-byte loads need
// element alignment only, which global memory allows: rows of any length and base stream alike.
typedef uint32_t raw4 __attribute__((ext_vector_type(4)));
typedef raw4 raw4_bf16 __attribute__((aligned(2)));
typedef raw4 raw4_f32 __attribute__((aligned(4)));

__device__ __forceinline__ void unpack_bf16(raw4 w, float (&x)[8]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) { x[2 * j] = bf16_lo(w[j]); x[2 * j + 1] = bf16_hi(w[j]); }
}

__device__ __forceinline__ void load8(const void* base, int dtype, int64_t row_off, int e0, int V, float (&x)[8]) {
  if (dtype == kBF16) {
    const uint16_t* p = static_cast<const uint16_t*>(base) + row_off;
    if (e0 + 8 <= V) {
      unpack_bf16(*reinterpret_cast<const raw4_bf16*>(p + e0), x);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (e0 + j < V) ? bf16_bits_to_float(p[e0 + j]) : -INFINITY;
    }
  } else {
    const float* p = static_cast<const float*>(base) + row_off;
    if (e0 + 8 <= V) {
      const raw4 a = *reinterpret_cast<const raw4_f32*>(p + e0);
      const raw4 b = *reinterpret_cast<const raw4_f32*>(p + e0 + 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) { x[j] = __uint_as_float(a[j]); x[4 + j] = __uint_as_float(b[j]); }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (e0 + j < V) ? p[e0 + j] : -INFINITY;
    }
  }
}

// N groups of eight logits with all their loads in flight together: no branch stands between one load and the next
// (a load inside a branch is waited for at the branch's end; the row statistics took four trips to memory for their
// four groups).  Group i holds the elements first8(e0[i], V) .. + 8 of its row: the last group of a row whose length
// eight does not divide starts earlier, and what lies ahead of e0[i] (or, for V < 8, at or beyond V) reads as -inf.
__device__ __forceinline__ int first8(int e0, int V) { return min(e0, max(V - 8, 0)); }

template <int DT, int N>
struct Raw8 {
  raw4 w[N][DT == kBF16 ? 1 : 2];
};
// DT: the matrix's dtype as a constant (with a branch on it the compiler merges the two sides' last loads through
// scratch memory).  row_off(i), e0(i): functions of the group number.
template <int DT, int N, typename Off, typename E0>
__device__ __forceinline__ void issue8(const void* base, Off row_off, E0 e0, int V, Raw8<DT, N>& r) {
  if (V < 8) return;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t at = row_off(i) + first8(e0(i), V);
    if constexpr (DT == kBF16) {
      r.w[i][0] = *reinterpret_cast<const raw4_bf16*>(static_cast<const uint16_t*>(base) + at);
    } else {
      r.w[i][0] = *reinterpret_cast<const raw4_f32*>(static_cast<const float*>(base) + at);
      r.w[i][1] = *reinterpret_cast<const raw4_f32*>(static_cast<const float*>(base) + at + 4);
    }
  }
}
// ... the values of group i (a constant after unrolling).  ROWS: the groups are of different rows; of one row only
// group 0 can start inside it when V < 8.
template <bool ROWS, int DT, int N>
__device__ __forceinline__ void take8(const void* base, int64_t row_off, int e0, int V, const Raw8<DT, N>& r, int i,
                                      float (&x)[8]) {
  if (V < 8) {
    if (ROWS || i == 0) {
      load8(base, DT, row_off, e0, V, x);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = -INFINITY;
    }
    return;
  }
  if constexpr (DT == kBF16) {
    unpack_bf16(r.w[i][0], x);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) { x[j] = __uint_as_float(r.w[i][0][j]); x[4 + j] = __uint_as_float(r.w[i][1][j]); }
  }
  if (__any(e0 > V - 8)) {
    const int skip = e0 - first8(e0, V);
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = j >= skip ? x[j] : -INFINITY;
  }
}

// Whole-wave reductions through the data-parallel-primitive path of the vector ALU (a few cycles per
// step, against a trip through the LDS crossbar per step for a shuffle): an inclusive scan inside
// each row of 16 lanes (row_shr 1, 2, 4, 8), then lane 15 of rows 0 and 2 is broadcast into rows 1 and 3
// (row_bcast:15) and lane 31 into rows 2 and 3 (row_bcast:31): an inclusive scan over the wave.  Lane 63 then holds
// the reduction, which is read back as a wave-uniform value.  Lanes without a source keep the identity.  All 64
// lanes have to be active.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double x) {
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROW_MASK, 0xf, false);
  hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROW_MASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_scan(double x) {
  x += dpp_f64<0x111, 0xf>(x);
  x += dpp_f64<0x112, 0xf>(x);
  x += dpp_f64<0x114, 0xf>(x);
  x += dpp_f64<0x118, 0xf>(x);
  x += dpp_f64<0x142, 0xa>(x);
  x += dpp_f64<0x143, 0xc>(x);
  return x;
}
__device__ __forceinline__ double lane_f64(double x, int lane) {        // lane: wave-uniform
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}
__device__ __forceinline__ double wave_sum(double x) { return lane_f64(wave_scan(x), 63); }
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max_step(float x) {
  const int ninf = 0xff800000;
  const int y = __builtin_amdgcn_update_dpp(ninf, __float_as_int(x), CTRL, ROW_MASK, 0xf, false);
  return fmaxf(x, __int_as_float(y));
}
__device__ __forceinline__ float wave_max(float x) {
  x = dpp_max_step<0x111, 0xf>(x);
  x = dpp_max_step<0x112, 0xf>(x);
  x = dpp_max_step<0x114, 0xf>(x);
  x = dpp_max_step<0x118, 0xf>(x);
  x = dpp_max_step<0x142, 0xa>(x);
  x = dpp_max_step<0x143, 0xc>(x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
// ... and over a row of 16 lanes, by rotations: the same bits in all 16.
__device__ __forceinline__ float row16_max(float x) {
  x = dpp_max_step<0x128, 0xf>(x);
  x = dpp_max_step<0x124, 0xf>(x);
  x = dpp_max_step<0x122, 0xf>(x);
  return dpp_max_step<0x121, 0xf>(x);
}
__device__ __forceinline__ double row16_sum(double x) {
  x += dpp_f64<0x128, 0xf>(x);
  x += dpp_f64<0x124, 0xf>(x);
  x += dpp_f64<0x122, 0xf>(x);
  return x + dpp_f64<0x121, 0xf>(x);
}

// Relaxed device-scope accesses: words that workgroups of one kernel exchange.
template <typename T> __device__ __forceinline__ T ld_dev(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void st_dev(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Messages between the workgroups of one launch: 64-bit words, 27 bits of data above the launch's 37-bit tag (next_message_tag
// in kernels.h).  Every word counts by itself, so that no order between words is needed.  An fp64 sum takes three words and
// leaves room for the upper half of an fp32 maximum, which is all of a maximum of bf16 logits; the lower half takes a
// fourth.  (40 bits of tag and four words whatever the logits, posted by one thread: 1 x 7 drafts x 128256 classes in one launch 12.1
// us, now 11.6, as with 32 bits of tag and three words, 11.8; 8 x 8 x 32000 behind the projection 11.8, now 11.6.)
constexpr int kTagBits = 37;
constexpr int kSumWords = 3, kRecordWords = 4;
constexpr int record_words(int dtype) { return dtype == kBF16 ? 3 : kRecordWords; }
template <int N>
__device__ __forceinline__ bool have_tag(const unsigned long long* w, unsigned long long tag) {      // all of w[0 .. N - 1]
  unsigned long long differ = w[0] ^ tag;
#pragma unroll
  for (int k = 1; k < N; ++k) differ |= w[k] ^ tag;
  return (differ << (64 - kTagBits)) == 0ull;
}
__device__ __forceinline__ unsigned long long message_word(int k, double z, float m, unsigned long long tag) {
  const unsigned lo = static_cast<unsigned>(__double2loint(z)), hi = static_cast<unsigned>(__double2hiint(z)), mb = __float_as_uint(m);
  unsigned d = lo;
  d = k == 1 ? (lo >> 27) | (hi << 5) : d;
  d = k == 2 ? (hi >> 22) | ((mb >> 16) << 10) : d;
  d = k == 3 ? mb & 0xffffu : d;
  return (static_cast<unsigned long long>(d) << kTagBits) | tag;
}
__device__ __forceinline__ double message_sum(const unsigned long long* w) {
  const unsigned d0 = static_cast<unsigned>(w[0] >> kTagBits), d1 = static_cast<unsigned>(w[1] >> kTagBits), d2 = static_cast<unsigned>(w[2] >> kTagBits);
  return __hiloint2double(static_cast<int>((d1 >> 5) | (d2 << 22)), static_cast<int>(d0 | (d1 << 27)));
}
template <int WORDS>
__device__ __forceinline__ float message_max(const unsigned long long* w) {
  unsigned m = static_cast<unsigned>(w[2] >> (kTagBits + 10)) << 16;
  if constexpr (WORDS > 3) m |= static_cast<unsigned>(w[3] >> kTagBits);
  return __uint_as_float(m);
}

// Per-(row, segment) softmax statistics written by the row-statistics kernel:
// m = largest logit of the segment (raw logit units, -inf if the segment is empty),
// z = sum over the segment of 2^((l - m) * c), c = log2(e)/T.
struct __align__(16) SegStat {
  float m;
  float pad;
  double z;
};

// (maximum, sum of 2^((l - max) c)) of a row over a workgroup's classes from those of its NW waves.
template <int NW>
__device__ __forceinline__ void merge_waves(const float* sh_m, const double* sh_z, float c, float& M, double& Z) {
  M = sh_m[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmaxf(M, sh_m[w]);
  Z = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (sh_m[w] != -INFINITY) Z += sh_z[w] * static_cast<double>(fast_exp2((sh_m[w] - M) * c));
}

// Merged (max, sum) of one logit row from its per-segment records load(0) .. load(nseg - 1), by a group of 16 lanes (lane sl
// of the group takes segments sl, sl + 16, ...); the result is in every lane of the group.  The arithmetic and its order
// are the same for every caller, so every caller gets the same bits (accept_walk_kernel merges by itself, in the
// order of its shuffles: equal up to the last bits).  All lanes of the wave take part
// (a group without a row passes nseg = 0).
template <typename Load>
__device__ __forceinline__ void merged_stats(Load load, int nseg, float c, int sl, float& m_out, double& z_out) {
  SegStat st;
  st.m = -INFINITY; st.pad = 0.f; st.z = 0.0;
  if (sl < nseg) st = load(sl);                    // up to 16 segments (131072 logits): one load per lane
  float m = st.m;
  for (int sg = sl + 16; sg < nseg; sg += 16) m = fmaxf(m, load(sg).m);
  m = row16_max(m);
  double z = 0.0;
  for (int sg = sl;;) {
    if (st.m != -INFINITY) z += st.z * exp2(static_cast<double>(st.m - m) * static_cast<double>(c));
    sg += 16;
    if (sg >= nseg) break;
    st = load(sg);
  }
  m_out = m;
  z_out = row16_sum(z);
}

// ... from records in memory.  DEV: read them with device-scope loads (they were written by other workgroups of the same
// kernel).
template <bool DEV>
__device__ __forceinline__ void merged_row_stats(const SegStat* __restrict__ rec, int nseg, float c, int sl,
                                                 float& m_out, double& z_out) {
  merged_stats([&](int sg) -> SegStat {
    if constexpr (DEV) {
      const unsigned long long* w = reinterpret_cast<const unsigned long long*>(rec + sg);
      const unsigned long long w0 = ld_dev(w), w1 = ld_dev(w + 1);
      SegStat st;
      st.m = __uint_as_float(static_cast<unsigned>(w0));
      st.pad = 0.f;
      st.z = __builtin_bit_cast(double, w1);
      return st;
    } else {
      return rec[sg];
    }
  }, nseg, c, sl, m_out, z_out);
}

}  // namespace specv
