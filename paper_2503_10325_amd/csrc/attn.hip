// Verify-attention for gfx950: the draft queries of each request attend over the paged
// bf16 KV cache (committed context + their draft ancestors), Section 2.1 / 4.2 of the
// paper (parallel verification with a tree-attention mask).
//
// Work decomposition.  All n*G query rows that share a KV head are processed together so every
// K/V byte is fetched once per KV head; long requests are cut into context chunks whose
// unnormalised partial results attn_combine_kernel merges (split-KV).  Two bodies:
//   token-split (stream_item, up to 64 query rows per KV head): a workgroup of 4 waves, or 8 where a
//     compute unit gets only one, per (request, KV head, chunk); every wave streams its own 32-token
//     tiles (2 cache pages) from memory straight to its private LDS tile, reads them as matrix operands
//     (V through transposing reads) and multiplies each with one or two 32-row query blocks; the waves
//     merge through LDS.
//   row-split (rows_item, more rows): the 4 or 8 waves of a workgroup stage 64-token tiles together
//     (double-buffered LDS: K straight from memory, V through registers, where it becomes fp16) and each
//     owns one block of 32 query rows.  Instantiated a second time for requests of 65 to 128 draft nodes (two ancestor-mask
//     words per node).
// Launches: attn_stream_kernel and attn_rows_kernel, grid-mapped, one body for the whole batch;
// attn_stream_list_kernel, ragged batches of up to 128 rows from a work list built on the device and
// sorted by length, and attn_mixed_kernel, such batches with little work: each request takes the body of
// its own row count.
// In both, S^T = K Q^T runs on v_mfma_f32_32x32x16_bf16 with the tokens as the M dimension, so
// each lane owns one query column and the online-softmax statistics need a single exchange
// between the half-waves.  V lies in LDS in natural rows; its operands come through transposing reads.
// O^T = V^T P^T: the token-split body keeps bf16 operands (weights as a high and a low bf16 term);
// the row-split body converts V to fp16 while staging it and uses fp16 weights in one
// v_mfma_f32_32x32x16_f16 term.
#include <stdlib.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace specv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = 4;
constexpr int kTile = 32;          // tokens per wave iteration
constexpr int kPage = 16;
constexpr int kMaxQ = 64;             // query nodes per request with one ancestor-mask word
constexpr int kMaxQWide = 128;        // ... with two (row-split kernels only)

template <int D>
struct AttnCfg {
  static constexpr int kCh = D / 8;                       // 16-byte chunks per token row
  static constexpr int kTokPerLoad = 64 / kCh;            // token rows one wave-wide load covers
  static constexpr int kQKSteps = D / 16;
  static constexpr int kDBlocks = D / 32;
  // token-split body: a wave's tile of K or V in LDS, natural token rows of kRowBytes without padding
  static constexpr int kRowBytes = D * 2;
  static constexpr int kPageBytes = kPage * kRowBytes;
  static constexpr int kPageLoads = kPageBytes / 1024;    // loads per page
  static constexpr int kTileBytes = kTile * kRowBytes;
  static constexpr int kQLdsFrags = kQKSteps + kQKSteps / 2;    // two query blocks per wave: 1 KB fragments kept in LDS
  // 16-byte chunk c of row r sits at position c ^ swizzle(r).  K operands: 16 rows at one chunk number in one go.  V: four
  // rows of 64 contiguous bytes.  Both spread over the 256 bytes that the LDS serves at a time.
  static __device__ constexpr int k_swizzle(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  static __device__ constexpr int v_swizzle(int r) { return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); }
  static constexpr int kORedStride = D + 4;               // floats; padded row of the cross-wave reduction
};

struct AttnParams {
  const uint16_t* q;
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  const int32_t* block_table;
  const int32_t* ctx_len;
  const int32_t* q_offsets;
  const int32_t* parent;
  void* out;
  float* lse;
  float* ws_o;       // [rows, max_chunks, D] unnormalised partial outputs
  float2* ws_ml;     // [rows, max_chunks] (max in log2 units, sum)
  int B, Hq, Hkv, G, max_pages, chunk_tokens, max_chunks;
  int tau;           // > 0: a request is cut so that one wave streams at most tau tiles per work item
  int tau_rows;      // ... of a request that runs the row-split body
  int list_rows_min; // > 0 (kernels with both bodies): requests with this many query rows per KV head use the row-split body
  int list_rows_units;        // sixteenths of a work-list unit that 32 tokens of such a request cost
  int chunks_last;            // grid-mapped token-split launch: blockIdx = (KV head, request, chunk)
  int xcd_swizzle;            // grid-mapped row-split launch: consecutive workgroups of the logical order share an XCD
  int n_cap;                  // query nodes per request the launched kernels handle (64, or 128 with two mask words)
  float c;           // scale * log2(e)
  int out_f32;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The value held by the same lane of the other half-wave (lane ^ 32), through the gfx950 half-wave
// swap instead of an LDS round trip: after swapping the upper half of one copy with the lower half
// of another, lane l of the first copy holds x[l % 32] and of the second x[32 + l % 32].
__device__ __forceinline__ void half_pair(float x, float& lo_half, float& hi_half) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo_half = __uint_as_float(r[0]);
  hi_half = __uint_as_float(r[1]);
}
__device__ __forceinline__ float half_max(float x) {
  float a, b;
  half_pair(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float half_sum(float x) {
  float a, b;
  half_pair(x, a, b);
  return a + b;
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ u32x4 zero4() {
  u32x4 z = {0u, 0u, 0u, 0u};
  return z;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Two fp32 values as two fp16 in one word (round toward zero: never rounds a finite value to infinity).
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}
// A word of two bf16 values as two fp16 values.  Exact for magnitudes in [2^-14, 65504] (bf16 carries 8
// significant bits, fp16 11); smaller magnitudes land on the fp16 subnormal grid (absolute error < 2^-24),
// larger ones saturate at 65504.
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t w) { return pack_f16(bf16_lo(w), bf16_hi(w)); }

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2 x = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, x);
}

// A zero the compiler cannot see through.  Added to the thread id at the top of a work item's body, it ties the
// per-lane constants of that body (lane offsets, LDS addresses) to the item: in a kernel that loops over items
// of two different bodies they would otherwise be hoisted out of the loop and held in registers across both.
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+s"(z));
  return z;
}

// 16 bytes per lane from base + off + 1024 j to LDS: lane i's land at byte lds_at + 1024 j + 16 i (the instruction's offset
// counts on both sides).  Not tracked by the compiler: the loops count these loads themselves (vmcnt).  The LDS address
// is an operand bound to M0: the compiler writes that register itself and knows when it changes.
__device__ __forceinline__ void load_to_lds(const unsigned char* base, unsigned off, unsigned lds_at, int j) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" :: "{m0}"(lds_at), "v"(off), "s"(base), "n"(1024 * j) : "memory");
}
__device__ __forceinline__ unsigned lds_address(unsigned char* p) {
  return static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)p));
}
__device__ __forceinline__ __attribute__((address_space(3))) u32x4* lds_u32x4(unsigned lds_at) {
  return (__attribute__((address_space(3))) u32x4*)lds_at;
}
typedef __attribute__((address_space(4))) int32_t const_i32;       // read through the scalar cache
// Which of 32 tokens a draft node sees that start at position p: bit i for token p + i, given left = ctx - p.  Context
// tokens all, drafts by the node's ancestor mask (which has no bit at or beyond the number of nodes).
__device__ __forceinline__ uint32_t tile_mask(unsigned long long anc, int left) {
  if (left >= 32) return 0xffffffffu;
  if (left > 0) return static_cast<uint32_t>(anc << left) | ((1u << left) - 1u);
  return left > -64 ? static_cast<uint32_t>(anc >> -left) : 0u;
}
// ... of a node with two mask words (up to 128 nodes), p being `past` >= 0 tokens behind the context.
__device__ __forceinline__ uint32_t wide_mask(unsigned long long lo, unsigned long long hi, int past) {
  if (past >= 128) return 0u;
  if (past >= 64) return static_cast<uint32_t>(hi >> (past - 64));
  const unsigned long long w = past == 0 ? lo : (lo >> past) | (hi << (64 - past));
  return static_cast<uint32_t>(w);
}
// Matrix operand of 8 tokens for this lane's head dimension from two transposing LDS reads of 4 tokens each.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ s16x4 tr_read(unsigned lds_at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)lds_at);
}
__device__ __forceinline__ bf16x8 tr_pair(unsigned p0, unsigned p1) {
  const s16x4 a = tr_read(p0), b = tr_read(p1);
  const s16x8 v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// Waves of a four-wave token-split workgroup that share the tiles of a request of R <= 128 query rows: all of them where a
// wave multiplies a tile with every query row (up to 64; short chunks aside, see stream_item), none where each has a 32-row block of its own.
__device__ __forceinline__ int stream_nslice(int R) {
  return R <= 64 ? 4 : 1;
}

// Kernels that hold both bodies run requests with at least P.list_rows_min query rows per KV head through the
// row-split body (its waves share every staged tile; the token-split body stages a tile once per 32-row block).
__device__ __forceinline__ bool list_uses_rows(const AttnParams& P, int n) {
  return P.list_rows_min > 0 && n * P.G >= P.list_rows_min;
}

// Length of a request in the work list's unit, the 32-token tiles one wave of the token-split body streams.
// A unit is 128 tokens of a request of up to 64 rows, whose four waves take a tile each.  For the row-split body 32 tokens
// count P.list_rows_units sixteenths of it (the host passes 5): ragged batches of 64 requests x 8 KV heads, 512 to 12587
// tokens, with 4/16, 5/16, 6/16 at 36 units per item: 80 rows 181 / 173 / 179 us, 128 rows 192 / 183 / 190.
__device__ __forceinline__ int request_units(const AttnParams& P, int L, int n) {
  const int tiles = (L + kTile - 1) / kTile;
  if (list_uses_rows(P, n)) return (tiles * P.list_rows_units + 15) / 16;
  const int nslice = stream_nslice(min(n * P.G, 128));
  return (tiles + nslice - 1) / nslice;
}

// Number of context chunks of a request with L tokens and n draft nodes.  The sorted work list (tau > 0) cuts by units, the
// other launches by tokens.  The attention kernels and the combine kernel all use this function.
__device__ __forceinline__ int request_chunks(const AttnParams& P, int L, int n) {
  const int tau = list_uses_rows(P, n) ? P.tau_rows : P.tau;
  if (P.tau > 0) return min(max(1, (request_units(P, L, n) + tau - 1) / tau), P.max_chunks);
  return min(max(1, (L + P.chunk_tokens - 1) / P.chunk_tokens), P.max_chunks);   // (the bound lengthens the chunks)
}

// Token-split body (up to 128 query rows per KV head and workgroup).  NW waves (4, or 8 in a workgroup that has a compute
// unit for itself) take 32-token tiles in turn; NQ: 32-row query blocks a wave multiplies every tile it streams with.
//   up to 32 rows  (NQ = 1): all waves share the one block, each streaming every NW-th tile;
//   up to 64 rows  (NQ = 2): the same, each wave with both blocks: no tile is fetched twice;
//                  (NQ = 1): half of the waves per block, each streaming every NW/2-th tile (repeats hit in L2); see stream_item;
//   more           (NQ = 1): one wave (NW = 8: two) per block, streaming every tile.
// One work item: (request b, KV head kvh, context chunk, row group rg).  Every return below is workgroup-uniform.
//
// A tile goes from memory to LDS directly (16 bytes per lane and load, no registers, no conversion) and natural token rows
// serve both products: K as it lies, V through transposing LDS reads.  The 16-byte chunks of a row are placed by XOR so
// that both reads spread over all banks.  K and V of the wave have one buffer each: the next tile's K goes out as soon as
// the scores have read this one's and travels under the softmax and the output product, V behind the output product.
template <int D, int NW, int NQ>
__device__ __forceinline__ void stream_tiles(const AttnParams& P, unsigned char* smem, int b, int kvh, int chunk, int rg,
                                             int q0, int n, int ctx, int nchunks, int cb) {
  using C = AttnCfg<D>;
  const int tid = static_cast<int>(threadIdx.x) + opaque_zero(), lane = tid & 63;
  __builtin_assume(tid >= 0 && tid < NW * kWave);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int L = ctx + n;
  const int R = n * P.G;
  const int row0 = rg * 128;
  const int nqb = min(4, (R - row0 + 31) / 32);             // query blocks of this workgroup
  const int groups = NQ == 2 || nqb == 1 ? 1 : (nqb == 2 ? 2 : 4);   // waves with tiles of their own come in so many kinds
  const int nslice = NW / groups;                           // waves sharing one query block
  const int my_g = wave % groups, my_slice = wave / groups;
  const bool wave_active = NQ * my_g < nqb;
  const int t_begin = chunk * cb;
  const int t_end = min(L, t_begin + cb);
  const int ntiles = (t_end - t_begin + kTile - 1) / kTile;

  unsigned char* k_lds = smem + wave * 2 * C::kTileBytes;
  unsigned char* v_lds = k_lds + C::kTileBytes;
  unsigned char* q_lds = smem + NW * 2 * C::kTileBytes;                                // query fragments (NQ = 2)
  unsigned long long* sh_anc = reinterpret_cast<unsigned long long*>(q_lds + C::kQLdsFrags * 1024);   // [64]
  int* sh_par = reinterpret_cast<int*>(sh_anc + kMaxQ);                                // [64]
  // the merge of the waves' results takes the tile memory
  float* sh_m = reinterpret_cast<float*>(smem + NW * 32 * C::kORedStride * sizeof(float));  // [NW][32]
  float* sh_l = sh_m + NW * 32;                                                        // [NW][32]

  // ---- tile loads: page ids come through scalar loads one tile ahead, a page of 16 token rows is contiguous ----
  const int64_t page_bytes = static_cast<int64_t>(P.Hkv) * kPage * C::kRowBytes;
  const unsigned char* k_head = reinterpret_cast<const unsigned char*>(P.k_pool) + static_cast<int64_t>(kvh) * kPage * C::kRowBytes;
  const unsigned char* v_head = reinterpret_cast<const unsigned char*>(P.v_pool) + static_cast<int64_t>(kvh) * kPage * C::kRowBytes;
  const const_i32* bt = (const const_i32*)(P.block_table + static_cast<int64_t>(b) * P.max_pages);
  const int last_page = (L - 1) / kPage;
  const unsigned lds_k = lds_address(k_lds), lds_v = lds_address(v_lds);
  // Ids past the request's last page repeat it, negative ids read page 0: the data is in bounds.
  int pg0 = 0, pg1 = 0;
  auto fetch_pages = [&](int t) {
    if (t < ntiles) {
      const int lp = (t_begin + kTile * t) / kPage;
      pg0 = max(bt[lp], 0);
      pg1 = max(bt[min(lp + 1, last_page)], 0);
    }
  };
  auto issue = [&](bool is_k) __attribute__((always_inline)) {        // of the tile whose page ids were fetched last
    const unsigned char* head = is_k ? k_head : v_head;
    int l = lane;
    asm volatile("" : "+v"(l));              // (worked out anew, as the operand addresses below: registers are what is short)
    const int row = l / C::kCh, ch = l % C::kCh;          // row and chunk of this lane within one load; load j: chunk ^ 4 j (K)
    const unsigned off = row * C::kRowBytes + ((ch ^ (is_k ? C::k_swizzle(row) : C::v_swizzle(row))) << 4);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const unsigned char* base = head + (p ? pg1 : pg0) * page_bytes;
#pragma unroll
      for (int j = 0; j < C::kPageLoads; ++j)
        load_to_lds(base, is_k ? off ^ (64u * j) : off, (is_k ? lds_k : lds_v) + p * C::kPageBytes, j);
    }
  };

  // Everything that depends on no other load goes out first - the page ids of the first tile, the query rows, the parents -
  // then the first tile's K and V; the masks are worked out while those are on their way.
  const bool touches_drafts = t_end > ctx;
  int t = my_slice;
  const bool any_tile = wave_active && t < ntiles;
  fetch_pages(t);
  // ---- this lane's query columns ----
  int node[NQ];
  auto q_ptr = [&](int qi, int& nd) {
    const int row = min(row0 + 32 * (NQ * my_g + qi) + ln, R - 1);     // (columns past the last row repeat it and are not written)
    nd = row / P.G;
    return P.q + (static_cast<int64_t>(q0 + nd) * P.Hq + kvh * P.G + row % P.G) * D + 8 * lh;
  };
  // NQ = 2: the second block, and the first steps of the first, are read from LDS by all waves (each wave brings its share
  // of the fragments there): what registers are left would not hold both blocks' accumulators and queries.
  constexpr int kQReg0 = NQ == 2 ? C::kQKSteps / 2 : 0;                      // first step that stays in registers
  constexpr int kQFrags = NQ == 2 ? C::kQLdsFrags : 0, kShare = (kQFrags + NW - 1) / NW;
  bf16x8 qf[C::kQKSteps];
  u32x4 q_share[kShare + 1];
  {
    const uint16_t* qp = q_ptr(0, node[0]);
#pragma unroll
    for (int ks = kQReg0; ks < C::kQKSteps; ++ks) qf[ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(qp + 16 * ks));
    if constexpr (NQ == 2) {
      const uint16_t* qp1 = q_ptr(1, node[1]);
#pragma unroll
      for (int i = 0; i < kShare; ++i) {
        const int f = min(wave + NW * i, kQFrags - 1);          // fragment: first block's first steps, then the second block's
        q_share[i] = *reinterpret_cast<const u32x4*>(f < kQReg0 ? qp + 16 * f : qp1 + 16 * (f - kQReg0));
      }
    }
  }
  // (here, where the page ids have to be waited for anyway: a value still on its way behind the tile's loads would be
  // waited for with all of them)
  if (touches_drafts && P.parent && tid < kMaxQ) sh_par[tid] = tid < n ? P.parent[q0 + tid] : -1;
  if (any_tile) {
    issue(true);
    issue(false);
    fetch_pages(t + nslice);
  }
  // operand reads: K, lane ln's row, 16-byte chunk 2 ks + lh at k_at ^ 32 ks (tiles start at multiples of 256 bytes); query
  // fragments as the lanes hold them
  const unsigned k_at = lds_k + ln * C::kRowBytes + ((lh ^ C::k_swizzle(ln)) << 4);
  const unsigned q_at = lds_address(q_lds) + 16 * lane;

  // ---- ancestor-or-self masks of the draft nodes (only chunks that reach the drafts) ----
  if (touches_drafts) {
    if (P.parent) __syncthreads();
    if (tid < kMaxQ) {
      unsigned long long mask = 0;
      if (tid < n) {
        if (P.parent) {
          int a = tid;
          for (int g = 0; g <= tid && a >= 0; ++g) {
            mask |= 1ull << a;
            const int p = sh_par[a];
            a = (p >= a || p < -1) ? -1 : p;
          }
        } else {
          mask = (2ull << tid) - 1ull;
        }
      }
      sh_anc[tid] = mask;
    }
  }
  if constexpr (NQ == 2) {
#pragma unroll
    for (int i = 0; i < kShare; ++i) *lds_u32x4(q_at + 1024 * min(wave + NW * i, kQFrags - 1)) = q_share[i];
  }
  if (touches_drafts || NQ == 2) __syncthreads();
  unsigned long long my_anc[NQ];
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi) my_anc[qi] = touches_drafts ? sh_anc[node[qi]] : 0ull;
  // the query rows are in registers before the loop: a wait for them inside it would wait for the tiles too
#pragma unroll
  for (int ks = kQReg0; ks < C::kQKSteps; ++ks) asm volatile("" :: "v"(qf[ks]));

  float m_run[NQ], l_run[NQ];
  f32x16 oacc[NQ][C::kDBlocks];
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi) {
    m_run[qi] = -INFINITY;
    l_run[qi] = 0.f;
#pragma unroll
    for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[qi][db][r] = 0.f;
  }
  // transposing reads of V: a group of 16 lanes gets a 4-token x 16-dimension piece, lane i of it dimension i.  Lane i
  // addresses four dimensions (i % 4) of token i / 4; the two halves of the wave take the tokens of the weights they hold.
  const int tr_tok = 4 * lh + ((lane & 15) >> 2);
  const unsigned v_at = lds_v + tr_tok * C::kRowBytes + 8 * (lane & 1) +
                        (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ C::v_swizzle(tr_tok)) << 4);

  for (; wave_active && t < ntiles; t += nslice) {
    const int tok0 = t_begin + kTile * t;
    const bool more = t + nslice < ntiles;

    // ---- S^T = K Q^T ----
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * C::kPageLoads) : "memory");          // K is here (V may still be on its way)
    f32x16 sacc[NQ];
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[qi][r] = 0.f;
    unsigned ka = k_at;
    asm volatile("" : "+v"(ka));
    auto k_frag = [&](int ks) __attribute__((always_inline)) { return *lds_u32x4(ka ^ (32 * ks)); };
    auto q_frag = [&](int f) __attribute__((always_inline)) { return *lds_u32x4(q_at + 1024 * f); };
    if constexpr (NQ == 1) {
      u32x4 kf[C::kQKSteps];
#pragma unroll
      for (int ks = 0; ks < C::kQKSteps; ++ks) kf[ks] = k_frag(ks);
#pragma unroll
      for (int ks = 0; ks < C::kQKSteps; ++ks)
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), qf[ks], sacc[0], 0, 0, 0);
    } else {
      // operands ahead of the products: K two steps, the queries one
      u32x4 kf[3], qa[2], qb[2];
      kf[0] = k_frag(0); qa[0] = q_frag(0); qb[0] = q_frag(kQReg0); kf[1] = k_frag(1);
#pragma unroll
      for (int ks = 0; ks < C::kQKSteps; ++ks) {
        __builtin_amdgcn_sched_barrier(0);
        if (ks + 1 < C::kQKSteps) qb[(ks + 1) % 2] = q_frag(kQReg0 + ks + 1);
        if (ks + 1 < kQReg0) qa[(ks + 1) % 2] = q_frag(ks + 1);
        if (ks + 2 < C::kQKSteps) kf[(ks + 2) % 3] = k_frag(ks + 2);
        const bf16x8 q0k = ks < kQReg0 ? as_bf16x8(qa[ks % 2]) : qf[ks];
        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks % 3]), q0k, sacc[0], 0, 0, 0);
        sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks % 3]), as_bf16x8(qb[ks % 2]), sacc[1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                               // K has been read
      issue(true);
    }

    // ---- mask, online softmax, P^T as two bf16 terms (value + rounding residual) ----
    // A single bf16 rounding of P (2^-9 relative) would dominate the output error; carrying the rounding residual in a
    // second bf16 term keeps ~16 bits of every weight.  The running maximum follows the true one exactly: the largest weight
    // of a row, which counts most, is then 1 and has no rounding error at all (followed only when it had grown by more than 8,
    // fp32 results were off by 2.4e-6 instead of 2.0e-6 of their 2-norm, and by two to three times as much at the worst).
    const bool need_mask = tok0 + kTile > ctx;
    u32x4 hi[NQ][2], lo[NQ][2];
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi) {
      float tmax = -INFINITY;
      if (need_mask) {
        // bit 8 (r / 4) + r % 4 of the lane's word: may the query see token tok0 + 4 lh + that bit
        uint32_t seen = tile_mask(my_anc[qi], ctx - tok0) >> (4 * lh);
        asm volatile("" : "+v"(seen));       // (stays behind the branch: worked out ahead of it, it would cost every tile)
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[qi][r] = (seen & (1u << (8 * (r >> 2) + (r & 3)))) ? sacc[qi][r] : -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[qi][r]);
      tmax *= P.c;                                   // c > 0: the maximum commutes with the scaling
      tmax = half_max(tmax);
      const float m_new = fmaxf(m_run[qi], tmax);
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = fast_exp2(m_run[qi] - m_safe);
      if (__any(alpha != 1.f)) {
#pragma unroll
        for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[qi][db][r] *= alpha;
      }
      float psum = 0.f;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float p0 = fast_exp2(fmaf(sacc[qi][8 * s + 2 * j], P.c, -m_safe));
          const float p1 = fast_exp2(fmaf(sacc[qi][8 * s + 2 * j + 1], P.c, -m_safe));
          psum += p0 + p1;
          const uint32_t h = pack_bf16(p0, p1);
          hi[qi][s][j] = h;
          lo[qi][s][j] = pack_bf16(p0 - bf16_lo(h), p1 - bf16_hi(h));
        }
      l_run[qi] = l_run[qi] * alpha + psum;
      m_run[qi] = m_new;
    }

    // ---- O^T += V^T P^T, 16 tokens at a time ----
    if (more) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * C::kPageLoads) : "memory");  // V is here (the next K may be on its way)
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (tok0 + kTile > L) {
      // last, partial tile: stale cache slots must not reach O (their weight is zero, zero times what they hold may not be)
      for (int i = (L - tok0) * C::kCh + lane; i < kTile * C::kCh; i += kWave) *reinterpret_cast<u32x4*>(v_lds + 16 * i) = zero4();
    }
    unsigned va = v_at;
    asm volatile("" : "+v"(va));
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db) {
        const unsigned at = (va ^ (64 * db)) + 16 * s * C::kRowBytes;
        const bf16x8 a = tr_pair(at, at + 8 * C::kRowBytes);
#pragma unroll
        for (int qi = 0; qi < NQ; ++qi) {
          oacc[qi][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(hi[qi][s]), oacc[qi][db], 0, 0, 0);
          oacc[qi][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(lo[qi][s]), oacc[qi][db], 0, 0, 0);
        }
      }
    if (more) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                               // V has been read
      issue(false);
      fetch_pages(t + 2 * nslice);
    }
  }

  // ---- merge the waves that share a query block, one block of each wave at a time ----
  float* sh_o = reinterpret_cast<float*>(smem);        // [NW waves][32][kORedStride]
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi) {
    l_run[qi] = half_sum(l_run[qi]);
    __syncthreads();                         // every wave is done with its tile memory (or with the block before)
    if (lane < 32) {
      sh_m[wave * 32 + lane] = m_run[qi];
      sh_l[wave * 32 + lane] = l_run[qi];
    }
    __syncthreads();
    float M = -INFINITY;
    for (int s = 0; s < nslice; ++s) M = fmaxf(M, sh_m[(my_g + groups * s) * 32 + ln]);
    const float fscale = (m_run[qi] == -INFINITY) ? 0.f : fast_exp2(m_run[qi] - M);
    if (wave_active) {
      // register 4a + c of block db: head dimension 32 db + 8 a + 4 lh + c
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          float* dst = sh_o + (wave * 32 + ln) * C::kORedStride + 32 * db + 8 * a + 4 * lh;
          *reinterpret_cast<float4*>(dst) = make_float4(oacc[qi][db][4 * a] * fscale, oacc[qi][db][4 * a + 1] * fscale,
                                                        oacc[qi][db][4 * a + 2] * fscale, oacc[qi][db][4 * a + 3] * fscale);
        }
    }
    __syncthreads();
    const int rn = (tid >> 3) & 31;                        // query column this thread finalises, of group tid / 256 on
    const int rd0 = (tid & 7) * (D / 8);                   // first of its D/8 dims
    for (int g = tid >> 8; g < groups; g += NW / 4) {
      const int orow = row0 + 32 * (NQ * g + qi) + rn;
      if (orow >= R) continue;
      float Mq = -INFINITY;
      for (int s = 0; s < nslice; ++s) Mq = fmaxf(Mq, sh_m[(g + groups * s) * 32 + rn]);
      float Ls = 0.f;
      float acc[D / 8];
#pragma unroll
      for (int i = 0; i < D / 8; ++i) acc[i] = 0.f;
      for (int s = 0; s < nslice; ++s) {
        const int w = g + groups * s;
        const float mw = sh_m[w * 32 + rn];
        if (mw != -INFINITY) Ls += sh_l[w * 32 + rn] * fast_exp2(mw - Mq);
#pragma unroll
        for (int i = 0; i < D / 8; i += 4) {
          const float4 v = *reinterpret_cast<const float4*>(sh_o + (w * 32 + rn) * C::kORedStride + rd0 + i);
          acc[i] += v.x; acc[i + 1] += v.y; acc[i + 2] += v.z; acc[i + 3] += v.w;
        }
      }
      const int onode = orow / P.G, og = orow % P.G;
      const int64_t grow = static_cast<int64_t>(q0 + onode) * P.Hq + kvh * P.G + og;
      if (nchunks == 1) {
        const float inv = 1.f / Ls;
        if (P.out_f32) {
          float* o = static_cast<float*>(P.out) + grow * D + rd0;
#pragma unroll
          for (int i = 0; i < D / 8; ++i) o[i] = acc[i] * inv;
        } else {
          uint32_t* o = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(P.out) + grow * D + rd0);
#pragma unroll
          for (int i = 0; i < D / 16; ++i) o[i] = pack_bf16(acc[2 * i] * inv, acc[2 * i + 1] * inv);
        }
        if (P.lse && (tid & 7) == 0) P.lse[grow] = (Mq + log2f(Ls)) * static_cast<float>(kLn2);
      } else {
        float* o = P.ws_o + (grow * P.max_chunks + chunk) * D + rd0;
#pragma unroll
        for (int i = 0; i < D / 8; ++i) o[i] = acc[i];
        if ((tid & 7) == 0) P.ws_ml[grow * P.max_chunks + chunk] = make_float2(Mq, Ls);
      }
    }
  }
}

// (q0, n, ctx: first query row, number of query nodes (already capped at kMaxQ) and context length of request b)
template <int D, int NW>
__device__ __forceinline__ void stream_item(const AttnParams& P, unsigned char* smem, int b, int kvh, int chunk, int rg,
                                            int q0, int n, int ctx) {
  if (n <= 0) return;
  const int L = ctx + n, left = n * P.G - rg * 128;         // query rows of this row group and behind
  if (left <= 0) return;
  const int nchunks = request_chunks(P, L, n);
  if (chunk >= nchunks) return;
  const int cb = (((L + nchunks - 1) / nchunks) + kTile - 1) & ~(kTile - 1);
  // Two blocks per wave save a fetch of every tile and cost a longer start (queries through LDS) and a second merge.  They pay
  // where the launch's tiles are many: more than three per wave and two workgroups per compute unit.  One block against two,
  // 40 or 64 rows, us, of 16, 120, 250, 375, 500, 900, 2000 tokens: 40 requests x 8 KV heads (four waves) 9.8 11.9 15.3 22.3 27.5 43.7
  // 86 against 9.8 12.9 16.4 22.3 26.9 41.1 76; 4 x 8 (eight waves) 8.2 8.4 9.6 12.0 13.5 16.3 18.3 against 9.5 10.1 11.3
  // 13.3 15.3 18.2 19.5.
  if constexpr (NW == 4) {
    if (left > 32 && left <= 64 && min(cb, L - chunk * cb) > 3 * NW * kTile)
      return stream_tiles<D, NW, 2>(P, smem, b, kvh, chunk, rg, q0, n, ctx, nchunks, cb);
  }
  stream_tiles<D, NW, 1>(P, smem, b, kvh, chunk, rg, q0, n, ctx, nchunks, cb);
}

// Grid-mapped launch: blockIdx = (chunk + max_chunks * row group, KV head, request) or, where the block table is much wider
// than the requests (P.chunks_last), (KV head, request, chunk); workgroups whose chunk does not exist return at once.  A
// workgroup takes its share of a compute unit's LDS whether it has work or not, so the many without then go last: 5
// requests x 4 KV heads with at most 6 chunks of the 16 launched 16.7 -> 12.1 us with the merge (11.8 with a table as wide
// as the longest request), 8 x 8 with 4 of 16 49.9 -> 29.4 (28.3).  Not always: the order puts the chunks of one request
// on few compute units (tight tables: 4 requests x 8 KV heads, mixed kernel, 24.7 -> 31.4 us; 64 x 8, six of 2500 tokens
// among short ones, 40.9 -> 51.2).
// NW = 8 (one workgroup per compute unit instead of two): for launches that have no second workgroup for a compute unit;
// twice the waves share a chunk's tiles, with no more chunks to merge.  1 request x 8 KV heads x 16000 tokens
// (56 rows, 512-token chunks) 25.6 -> 24.6 us with the merge, 8 x 32 x 2048 46.0 -> 45.3.
template <int D, int NW>
__global__ __launch_bounds__(NW * kWave, NW == 4 ? 2 : 1) void attn_stream_kernel(AttnParams P) {
  extern __shared__ __align__(256) unsigned char smem[];
  const int b = P.chunks_last ? blockIdx.y : blockIdx.z, kvh = P.chunks_last ? blockIdx.x : blockIdx.y;
  const int cut = P.chunks_last ? blockIdx.z : blockIdx.x;
  const int q0 = P.q_offsets[b];
  int n = P.q_offsets[b + 1] - q0;
  n = n > kMaxQ ? kMaxQ : n;
  stream_item<D, NW>(P, smem, b, kvh, cut % P.max_chunks, cut / P.max_chunks, q0, n, P.ctx_len[b]);
}

constexpr int kPlanMaxB = 128;

// ----------------------------------------------------------------------------------
// Row-split variant for requests with more than 64 query rows per KV head (GQA groups
// times several drafts, draft trees).  The NW waves of a workgroup stage 64-token tiles
// cooperatively (double-buffered in LDS) and every wave owns one block of 32 query rows,
// for which it sees every token: no cross-wave merge is needed.
// K of the next tile goes to LDS directly; V of the next tile is converted ahead of the matrix instructions of the
// scores, stored between them, and needs no transposition (218 -> 165 vector instructions per wave
// and tile against staging both through registers and packing V with v_perm).  What bounds it is the issue of vector and matrix
// instructions of the two waves of a SIMD, which add up more than they overlap, and, with the tables in HBM, the clock: with
// L2-resident tables 64 x 8 KV heads x 2048 tokens x 128 rows 86.5 -> 80.1 us, 16 x 8 x 4096 x 256 rows 88.7 -> 84.6, 464 rows
// 138 -> 131; 256 rows from HBM 94.9 -> 91.0 in a step; short contexts gain the most (512 tokens, 160 rows 17.1 -> 14.3).
// One page id and one scalar base per wave and tile, and operand reads that need no address arithmetic (RowsCfg): about 500
// -> 410 instructions per wave and step of the sliced kernel.  In loops of the attention call, tables from HBM: 16 x 8 KV heads x
// 4096 tokens x 256 rows 95.7 -> 90.3 us, 464 rows 150.8 -> 148.3, 32 x 8 x 2048 x 224 85.4 -> 83.2, 64 x 8 x 2048 x 240
// 177.6 -> 175.1, ragged 64 x 8, 16 to 80 rows 173.7 -> 170.8.  (The conversion of V stands ahead of the scores' matrix
// instructions, where the compiler puts it: pinned between them the first of these takes 95.)
// ----------------------------------------------------------------------------------
// SL = 2 ("sliced"): the workgroup owns 32 * NW / 2 query rows and stages 128-token tiles; waves w and w + NW/2
// share a block of 32 rows, the first computing the lower 64 tokens of every staged tile, the second the upper 64,
// and they merge their results through LDS at the end.  It fills the chip from half as many (request, KV head,
// 256-row group) triples as SL = 1 without cutting the context (no partial results in memory, no combine kernel).
template <int D, int NW, int SL = 1>
struct RowsCfg {
  static constexpr int kTc = 64;                           // tokens one wave computes per step
  static constexpr int kT = kTc * SL;                      // tokens per staged tile
  static constexpr int kThreads = NW * 64;
  static constexpr int kTpt = kT * (D / 8) / kThreads;     // 16-byte loads per thread and tensor: consecutive tokens of V
  static constexpr int kTileBytes = kT * D * 2;            // bytes of a tile: natural rows, chunks placed by XOR as in the token-split body
  static constexpr int kStage = 2 * kTileBytes;            // K as bf16, V as fp16
  // The two tiles of K lie side by side, the two of V behind them: what an operand read adds to its lane's address, the stage
  // among it, then fits the 16 bits an LDS instruction has for it (with K and V of a stage side by side the tiles of 128
  // tokens took an addition per read in every second step).
  static constexpr int kV0 = 2 * kTileBytes;
  static_assert(kTileBytes + 64 * D * 2 <= 65536, "stage and row offsets of an operand read within an instruction's offset");
  static constexpr int kMaxChunkPages = NW == 8 ? 1024 : 512;   // a chunk spans at most 16384 (8192) tokens
  static constexpr int kPagePad = 32;                      // page-table entries kept past a chunk's last page
  // behind the two stages: ancestor masks, parents, page table
  static constexpr int meta_bytes(bool wide) { return wide ? kMaxQWide * 16 + kMaxQWide * 4 : kMaxQ * 8 + kMaxQ * 4; }
  static constexpr int lds_bytes(bool wide) { return 2 * kStage + meta_bytes(wide) + (kMaxChunkPages + kPagePad) * 4; }
  static constexpr int kLds = lds_bytes(false);
  static constexpr int kPageLoads = AttnCfg<D>::kPageLoads;
  static_assert(kTpt == 4 || kTpt == 2, "unsupported tile/thread combination");
  static_assert(kPageLoads % kTpt == 0, "a wave's loads of a tile are of one page");
};

// One work item of the row-split body: (request b, KV head kvh, context chunk `chunk` of `nchunks`, row group
// rg).  The request's context is cut into nchunks pieces of cb tokens (a multiple of the tile).  Every return
// below is workgroup-uniform up to the last barrier.
// WIDE: up to 128 query nodes per request (two mask words per node) instead of 64.  SL: see RowsCfg.
template <int D, int NW, bool WIDE = false, int SL = 1>
__device__ __forceinline__ void rows_item(const AttnParams& P, unsigned char* smem, int b, int kvh, int chunk, int rg,
                                          int nchunks, int cb, int q0, int n, int ctx) {
  using C = AttnCfg<D>;
  using RC = RowsCfg<D, NW, SL>;
  constexpr int kRowWaves = NW / SL;            // waves with row blocks of their own
  const int tid = static_cast<int>(threadIdx.x) + opaque_zero(), lane = tid & 63, wave = tid >> 6;
  __builtin_assume(tid >= 0 && tid < RC::kThreads);
  const int ln = lane & 31, lh = lane >> 5;

  if (n <= 0) return;
  const int L = ctx + n;
  const int R = n * P.G;
  const int row0 = rg * (32 * kRowWaves);
  if (row0 >= R) return;
  if (chunk >= nchunks) return;
  const int t_begin = chunk * cb;
  if (t_begin >= L) {                           // rounding the chunk up to whole tiles can empty the last one
    for (int r = row0 + tid; r < min(R, row0 + 32 * kRowWaves); r += RC::kThreads) {
      const int64_t g = static_cast<int64_t>(q0 + r / P.G) * P.Hq + kvh * P.G + r % P.G;
      P.ws_ml[g * P.max_chunks + chunk] = make_float2(-INFINITY, 0.f);
    }
    return;
  }
  const int t_end = min(L, t_begin + cb);
  const int ntiles = (t_end - t_begin + RC::kT - 1) / RC::kT;

  constexpr int kNodes = WIDE ? kMaxQWide : kMaxQ;
  constexpr int kWords = WIDE ? 2 : 1;
  unsigned long long* sh_anc = reinterpret_cast<unsigned long long*>(smem + 2 * RC::kStage);          // [kNodes][kWords]
  int* sh_par = reinterpret_cast<int*>(smem + 2 * RC::kStage + kNodes * kWords * 8);                  // [kNodes]
  int* sh_pages = reinterpret_cast<int*>(smem + 2 * RC::kStage + RC::meta_bytes(WIDE));               // [kMaxChunkPages]

  // Everything that depends on no other load goes out first (parents, query rows, the chunk's page ids), then the first
  // tile's K and V; the masks are worked out while those are on their way.
  const bool touches_drafts = t_end > ctx;
  int my_par = -1;
  if (touches_drafts && P.parent && tid < n) my_par = P.parent[q0 + tid];
  // ---- this wave's 32 query rows ----
  const int slice = SL == 1 ? 0 : wave / kRowWaves;          // which 64 tokens of a staged tile this wave computes
  const int wrow0 = row0 + 32 * (wave % kRowWaves);
  const bool active = wrow0 < R;                // wave-uniform
  const int row = wrow0 + ln;
  const bool valid = row < R;
  const int node = valid ? row / P.G : 0;
  const int gq = valid ? row % P.G : 0;
  const int64_t grow = static_cast<int64_t>(q0 + node) * P.Hq + kvh * P.G + gq;
  bf16x8 qf[C::kQKSteps];
  {
    const uint16_t* qp = P.q + grow * D + 8 * lh;
#pragma unroll
    for (int ks = 0; ks < C::kQKSteps; ++ks) {
      u32x4 v = zero4();
      if (valid) v = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
      qf[ks] = as_bf16x8(v);
    }
  }
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 oacc[C::kDBlocks];
#pragma unroll
  for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;

  // ---- cooperative tile loads ----
  const int32_t* bt = P.block_table + static_cast<int64_t>(b) * P.max_pages;
  const int vc = tid % C::kCh;                  // V: 16-byte chunk of the token row
  const int vtok0 = tid / C::kCh * RC::kTpt;    // V: first of kTpt consecutive tokens within the tile
  // two register sets for V: while tile t is computed, tile t+1 is converted and stored from one and tile t+2 is in flight
  // into the other (a third for tile t+3 with the loads at the top: 100.7 -> 108 us)
  u32x4 vrA[RC::kTpt], vrB[RC::kTpt];

  // Page ids of the whole chunk go to LDS once, so that the tile loads depend on no global read.
  const int lp0 = t_begin / kPage;
  const int np = (t_end + kPage - 1) / kPage - lp0;          // >= 1 pages touched by this chunk
  // (entries past the chunk's last page repeat it: tile numbers past the end need no clamp)
  for (int i = tid; i < np + RC::kPagePad; i += RC::kThreads) sh_pages[i] = max(bt[lp0 + min(i, np - 1)], 0);
  if (tid < kNodes) sh_par[tid] = my_par;
  __syncthreads();

  // Loads are unconditional (addresses clamped to the chunk's last page): positions past the end are masked out of the
  // scores, and their V values are zeroed when staged.  A wave's share of a tile, K and V alike, is kTpt loads within one cache
  // page: one page id, one scalar base (32 x 32 bits: pages and page sizes are not negative), a small per-lane offset; the
  // loads differ by the instruction's offset.  K goes from memory straight to LDS, the tokens from 16 wave_page + kTokPerLoad part0 on.
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  const int wave_page = uwave * RC::kTpt / RC::kPageLoads, part0 = uwave * RC::kTpt % RC::kPageLoads;
  const int k_row = lane / C::kCh, k_ch = lane % C::kCh;
  const unsigned k_lane_off = (k_row * C::kRowBytes + ((k_ch ^ C::k_swizzle(k_row)) << 4)) ^ (64u * part0);
  const unsigned v_lane_off = (vtok0 % kPage) * C::kRowBytes + vc * 16;
  const unsigned lds0 = lds_address(smem);
  const unsigned k_dst = lds0 + 1024 * RC::kTpt * uwave;
  const unsigned page_bytes = static_cast<unsigned>(P.Hkv) * (kPage * C::kRowBytes);
  const int64_t head_off = static_cast<int64_t>(kvh) * (kPage * C::kRowBytes);
  const unsigned char* k_base = reinterpret_cast<const unsigned char*>(P.k_pool) + head_off + part0 * 1024;
  const unsigned char* v_base = reinterpret_cast<const unsigned char*>(P.v_pool) + head_off;
  // The page ids of a tile are read from LDS a whole tile step before the loads that need them.
  int pk, pv;
  auto tile_page = [&](int t) { return sh_pages[min(RC::kT * t / kPage, np + RC::kPagePad - RC::kT / kPage) + wave_page]; };
  auto fetch_k_page = [&](int t) { pk = tile_page(t); };
  auto fetch_v_page = [&](int t) { pv = tile_page(t); };
  auto page_at = [&](const unsigned char* base, int page) __attribute__((always_inline)) {
    return base + static_cast<uint64_t>(static_cast<unsigned>(__builtin_amdgcn_readfirstlane(page))) * page_bytes;
  };
  auto issue_k = [&](int stage) __attribute__((always_inline)) {          // of the tile whose K page was fetched last
    const unsigned char* base = page_at(k_base, pk);
#pragma unroll
    for (int j = 0; j < RC::kTpt; ++j) load_to_lds(base, k_lane_off ^ (64u * j), k_dst + stage * RC::kTileBytes, j);
  };
  auto issue_v = [&](u32x4 (&vr)[RC::kTpt]) __attribute__((always_inline)) {
    const uint16_t* vp = reinterpret_cast<const uint16_t*>(page_at(v_base, pv) + v_lane_off);
#pragma unroll
    for (int i = 0; i < RC::kTpt; ++i) vr[i] = *reinterpret_cast<const u32x4*>(vp + i * D);
  };
  auto arrived = [&](u32x4 (&vr)[RC::kTpt]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < RC::kTpt; ++i) asm volatile("" : "+v"(vr[i]));
  };
  // never multiply stale cache slots (past ctx+n) into O: stage them as zeros
  auto cut_tail = [&](int t, u32x4 (&vr)[RC::kTpt]) {
    if (t_begin + RC::kT * (t + 1) > L) {                     // only the last tile (and the ones past it)
      const int left = L - (t_begin + RC::kT * t + vtok0);    // tokens of this thread that exist
#pragma unroll
      for (int i = 0; i < RC::kTpt; ++i)
        if (i >= left) vr[i] = zero4();
    }
  };
  // V goes to LDS as fp16 (the weights P are fp16 too: 11 significant bits in ONE matrix term), in natural rows: the
  // operand reads transpose.
  auto convert = [&](u32x4& v, int from) __attribute__((always_inline)) {
    v[from] = bf16x2_to_f16x2(v[from]);
    v[from + 1] = bf16x2_to_f16x2(v[from + 1]);
  };
  const unsigned v_store = lds0 + RC::kV0 + vtok0 * C::kRowBytes;
  auto store_v = [&](int stage, int i, const u32x4& v) __attribute__((always_inline)) {
    *lds_u32x4(v_store + stage * RC::kTileBytes + i * C::kRowBytes + ((vc ^ C::v_swizzle((vtok0 + i) & 3)) << 4)) = v;
  };

  unsigned long long my_anc = 0ull, my_anc_hi = 0ull;          // ancestor mask of this lane's node (set below)

  // One 64-token tile = one online-softmax step in two parts (scores, output) that share these registers.
  f32x16 sacc[2];
  f16x8 ph, va[C::kDBlocks];
  float m_safe = 0.f, m_next = -INFINITY, alpha = 1.f, psum = 0.f;
  // transposing reads, as in the token-split body: lane i of a group of 16 gets head dimension i of 4 tokens
  const int tr_tok = 4 * lh + ((lane & 15) >> 2);
  const unsigned v_at = lds0 + RC::kV0 + (RC::kTc * slice + tr_tok) * C::kRowBytes + 8 * (lane & 1) +
                        (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ C::v_swizzle(tr_tok)) << 4);
  auto v_frag = [&](int stage, int chunk, int db) {      // chunk = 16-token group 0..3 of the tile
    const unsigned at = (v_at ^ (64u * db)) + stage * RC::kTileBytes + 16 * chunk * C::kRowBytes;
    return __builtin_bit_cast(f16x8, tr_pair(at, at + 8 * C::kRowBytes));
  };
  const unsigned k_at = lds0 + (RC::kTc * slice + ln) * C::kRowBytes + ((lh ^ C::k_swizzle(ln)) << 4);
  // P^T as fp16 (weights lie in [0, 2^8]: 11 significant bits, against 8 of bf16, keep the output's error at the
  // level of its own bf16 rounding with a single matrix term), 16 tokens at a time
  auto p_chunk = [&](int chunk, f16x8& dst) __attribute__((always_inline)) {
    const int tb = chunk >> 1, sg = chunk & 1;
    u32x4 hw;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float p0 = fast_exp2(fmaf(sacc[tb][8 * sg + 2 * j], P.c, -m_safe));
      const float p1 = fast_exp2(fmaf(sacc[tb][8 * sg + 2 * j + 1], P.c, -m_safe));
      psum += p0 + p1;
      hw[j] = pack_f16(p0, p1);
    }
    dst = __builtin_bit_cast(f16x8, hw);
  };

  // First half: S = K Q^T (operand reads from LDS run two steps ahead of the matrix instructions that consume
  // them), with the stores of the next tile's V between the matrix instructions; mask, row maxima, rescale, the weights of the
  // first 16 tokens.
  auto tile_scores = [&](int stage, int t, u32x4 (&vr)[RC::kTpt]) __attribute__((always_inline)) {
    const int tok0 = t_begin + RC::kT * t + RC::kTc * slice;
    auto k_frag = [&](int ks, int tb) {
      return as_bf16x8(*lds_u32x4((k_at ^ (32 * ks)) + stage * RC::kTileBytes + 32 * tb * C::kRowBytes));
    };
    constexpr int kHalves = 2 * RC::kTpt;         // half rows of V to convert
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[tb][r] = 0.f;
    // three operand slots in rotation: the slot refilled at step ks was last read by the MFMAs
    // of step ks-1, never by the ones just issued
    bf16x8 ka[3][2];
    ka[0][0] = k_frag(0, 0); ka[0][1] = k_frag(0, 1);
    ka[1][0] = k_frag(1, 0); ka[1][1] = k_frag(1, 1);
#pragma unroll
    for (int ks = 0; ks < C::kQKSteps; ++ks) {
      __builtin_amdgcn_sched_barrier(0);
      if (ks + 2 < C::kQKSteps) {
        ka[(ks + 2) % 3][0] = k_frag(ks + 2, 0);
        ka[(ks + 2) % 3][1] = k_frag(ks + 2, 1);
      }
      sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks % 3][0], qf[ks], sacc[0], 0, 0, 0);
      sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks % 3][1], qf[ks], sacc[1], 0, 0, 0);
#pragma unroll
      for (int h = ks * kHalves / C::kQKSteps; h < (ks + 1) * kHalves / C::kQKSteps; ++h) {
        convert(vr[h / 2], 2 * (h & 1));
        if (h & 1) store_v(stage ^ 1, h / 2, vr[h / 2]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // V^T operand of the first 16 tokens is fetched while the scores are reduced
#pragma unroll
    for (int db = 0; db < C::kDBlocks; ++db) va[db] = v_frag(stage, 0, db);

    if (tok0 + RC::kTc > ctx) {                  // tile reaches the drafts or the end: apply the mask
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const int left = ctx - tok0 - 32 * tb;
        uint32_t seen = tile_mask(my_anc, left);
        if constexpr (WIDE) {
          if (left <= 0) seen = wide_mask(my_anc, my_anc_hi, -left);
        }
        seen >>= 4 * lh;
        asm volatile("" : "+v"(seen));
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[tb][r] = (seen & (1u << (8 * (r >> 2) + (r & 3)))) ? sacc[tb][r] : -INFINITY;
      }
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[tb][r]);
    tmax *= P.c;                                   // c > 0: the maximum commutes with the scaling
    tmax = half_max(tmax);
    // The running maximum only has to bound the exponents: it follows the true maximum when that is first
    // finite or has grown by more than 8 (weights then reach 2^8 at most, exact in fp16 and fp32); the
    // accumulator is rescaled on those steps alone, and the final O / l is the same quotient either way.
    m_next = fmaxf(m_run, tmax);
    if (m_run != -INFINITY && tmax <= m_run + 8.f) m_next = m_run;
    m_safe = (m_next == -INFINITY) ? 0.f : m_next;
    alpha = fast_exp2(m_run - m_safe);
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
    }
    psum = 0.f;
    p_chunk(0, ph);
  };

  // Second half: O += P V, 16 tokens at a time, with the exponentials of the next 16 tokens between the
  // matrix instructions of the current ones.
  auto tile_output = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int chunk = 0; chunk < 4; ++chunk) {
      __builtin_amdgcn_sched_barrier(0);
      f16x8 vn[C::kDBlocks];
      f16x8 nh;
      if (chunk + 1 < 4) {
#pragma unroll
        for (int db = 0; db < C::kDBlocks; ++db) vn[db] = v_frag(stage, chunk + 1, db);
      }
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db)
        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[db], ph, oacc[db], 0, 0, 0);
      if (chunk + 1 < 4) {
        p_chunk(chunk + 1, nh);
        // A wave issues in order: matrix instructions queued back to back would hold the weights of the next
        // 16 tokens behind them.  One matrix instruction, one operand read, then a quarter of the vector work.
#pragma unroll
        for (int i = 0; i < C::kDBlocks; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
        }
        ph = nh;
#pragma unroll
        for (int db = 0; db < C::kDBlocks; ++db) va[db] = vn[db];
      }
    }
    l_run = l_run * alpha + psum;
    m_run = m_next;
  };

  // ---- pipeline: while tile t is computed from one stage, V of tile t+1 is converted and stored to the other, K of tile t+1
  // travels to it, and V of the tiles behind travels to registers ----
  // Loads are issued unconditionally, also for tile numbers past the end (their addresses are clamped to the chunk's last
  // page, their V rows staged as zeros, and they are never computed): every path leaves the same number outstanding.
  // (a wave of the sliced variant skips a staged tile whose half for it lies past the end)
  auto mine = [&](int t) { return active && t < ntiles && t_begin + RC::kT * t + RC::kTc * slice < t_end; };
  fetch_k_page(0);
  fetch_v_page(0);
  issue_v(vrA);
  issue_k(0);
  fetch_k_page(1);
  fetch_v_page(1);
  if (touches_drafts) {
    if (tid < kNodes) {
      unsigned long long mask = 0, mask_hi = 0;
      if (tid < n) {
        if (P.parent) {
          int a = tid;
          for (int g = 0; g <= tid && a >= 0; ++g) {
            if (WIDE && a >= 64) mask_hi |= 1ull << (a - 64);
            else mask |= 1ull << a;
            const int p = sh_par[a];
            a = (p >= a || p < -1) ? -1 : p;
          }
        } else if (WIDE && tid >= 64) {
          mask = ~0ull;
          mask_hi = (2ull << (tid - 64)) - 1ull;
        } else {
          mask = (2ull << tid) - 1ull;
        }
      }
      sh_anc[tid * kWords] = mask;
      if (WIDE) sh_anc[tid * kWords + 1] = mask_hi;
    }
    __syncthreads();
  }
  if (touches_drafts && valid) {
    my_anc = sh_anc[node * kWords];
    if (WIDE) my_anc_hi = sh_anc[node * kWords + 1];
  }
  // (K of the tile that is computed next is here, this wave's part of its V is stored; the kTpt loads of V behind it are not waited for)
  auto stage_done = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(RC::kTpt) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto stage_v = [&](int stage, u32x4 (&vr)[RC::kTpt]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < RC::kTpt; ++i) { convert(vr[i], 0); convert(vr[i], 2); store_v(stage, i, vr[i]); }
  };
  arrived(vrA);
  cut_tail(0, vrA);
  stage_v(0, vrA);
  issue_v(vrB);
  fetch_v_page(2);
  issue_v(vrA);
  fetch_v_page(3);
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(2 * RC::kTpt) : "memory");       // K of the first tile
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  // V of tile t+1 has been in flight to `cur`, V of tile t+2 is to the other set, V of tile t+3 follows to `cur` when this wave
  // is done with tile t.  K of tile t+1 goes out at the top or, where one workgroup has the compute unit, behind the scores:
  // the waves come there one after the other, at the top the loads of all of them are one burst (256 rows x 4096 tokens, from
  // HBM in a step: 100.7 us with K and V at the top, 96.3 with K, 94.0 with half of K, 91.0 behind the scores).  Two workgroups
  // of four waves are out of step by themselves, and behind the scores is late for them (80 rows, work list 144 -> 155).
  constexpr bool kLateK = NW == 8;
  auto step = [&](int t, int stage, u32x4 (&cur)[RC::kTpt]) __attribute__((always_inline)) {
    arrived(cur);
    if constexpr (!kLateK) { issue_k(stage ^ 1); fetch_k_page(t + 2); }
    cut_tail(t + 1, cur);
    const bool work = mine(t);
    if (work) tile_scores(stage, t, cur);
    else stage_v(stage ^ 1, cur);
    if constexpr (kLateK) { issue_k(stage ^ 1); fetch_k_page(t + 2); }
    if (work) tile_output(stage);
    issue_v(cur);
    fetch_v_page(t + 4);
    stage_done();
  };
  for (int t = 0; t < ntiles; t += 2) {
    step(t, 0, vrB);
    step(t + 1, 1, vrA);
  }

  l_run = half_sum(l_run);
  if constexpr (SL == 2) {
    // ---- the wave that took the upper halves of the tiles hands (m, l, O) to the one that took the lower halves
    // (the tile memory is free: the loop ended with a barrier); accumulator registers go over as they are, one
    // 256-byte row of LDS per register ----
    float* xo = reinterpret_cast<float*>(smem) + (wave % kRowWaves) * (C::kDBlocks * 16 + 2) * 64;
    if (slice == 1 && active) {
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) xo[(db * 16 + r) * 64 + lane] = oacc[db][r];
      xo[(C::kDBlocks * 16) * 64 + lane] = m_run;
      xo[(C::kDBlocks * 16 + 1) * 64 + lane] = l_run;
    }
    __syncthreads();
    if (slice == 1) return;
    if (active) {
      const float m2 = xo[(C::kDBlocks * 16) * 64 + lane], l2 = xo[(C::kDBlocks * 16 + 1) * 64 + lane];
      const float M = fmaxf(m_run, m2);
      const float f1 = m_run == -INFINITY ? 0.f : fast_exp2(m_run - M);
      const float f2 = m2 == -INFINITY ? 0.f : fast_exp2(m2 - M);
#pragma unroll
      for (int db = 0; db < C::kDBlocks; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = oacc[db][r] * f1 + xo[(db * 16 + r) * 64 + lane] * f2;
      l_run = l_run * f1 + l2 * f2;
      m_run = M;
    }
  }
  // ---- write this wave's rows ----
  if (!active) return;
  if (!valid) return;
  // The weights were truncated to fp16 (round toward zero): every one is low by a factor that is uniform in
  // [0, 2^-11], 2^-12 on average, while the denominator l was summed from the unrounded weights.  The
  // average is put back here; what remains is the zero-mean part (2^-12 at most per weight).
  constexpr float kRtzFix = 1.f + 1.f / 4096.f;
  // register 4a + c of block db: head dimension 32 db + 8 a + 4 lh + c
  const float oscale = nchunks == 1 ? kRtzFix / l_run : kRtzFix;
  float* part = P.ws_o + (grow * P.max_chunks + chunk) * D;
#pragma unroll
  for (int db = 0; db < C::kDBlocks; ++db) {
    if (nchunks != 1 || P.out_f32) {
      // fp32 rows: the two halves of the wave write 32 contiguous bytes per row
      float* o = (nchunks != 1 ? part : static_cast<float*>(P.out) + grow * D) + 32 * db + 4 * lh;
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<float4*>(o + 8 * a) = make_float4(oacc[db][4 * a] * oscale, oacc[db][4 * a + 1] * oscale,
                                                            oacc[db][4 * a + 2] * oscale, oacc[db][4 * a + 3] * oscale);
    } else {
      // bf16 rows: the halves exchange their four dimensions of blocks a and a + 1, each then writes eight
#pragma unroll
      for (int a = 0; a < 4; a += 2) {
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t x = pack_bf16(oacc[db][4 * a + 2 * i] * oscale, oacc[db][4 * a + 2 * i + 1] * oscale);
          const uint32_t y = pack_bf16(oacc[db][4 * a + 4 + 2 * i] * oscale, oacc[db][4 * a + 5 + 2 * i] * oscale);
          const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
          o[i] = r[0];
          o[2 + i] = r[1];
        }
        *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(P.out) + grow * D + 32 * db + 8 * (a + lh)) = o;
      }
    }
  }
  if (nchunks == 1) {
    if (P.lse && lh == 0) P.lse[grow] = (m_run + log2f(l_run)) * static_cast<float>(kLn2);
  } else if (lh == 0) {
    P.ws_ml[grow * P.max_chunks + chunk] = make_float2(m_run, l_run);
  }
}

template <int D, int NW, bool WIDE, int SL>
__global__ __launch_bounds__(NW * 64, (NW == 4 ? 2 : 1)) void attn_rows_kernel(AttnParams P) {
  extern __shared__ __align__(256) unsigned char smem[];
  unsigned bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (P.xcd_swizzle) {
    // Workgroups go to the 8 XCDs in turn.  With several row groups per (request, KV head) pair, renumber so that
    // the row groups of a pair run on one XCD at the same time: the second read of the pair's K/V hits in that L2.
    const unsigned total = gridDim.x * gridDim.y * gridDim.z;           // a multiple of 8 (checked by the host)
    const unsigned linear = bx + gridDim.x * (by + gridDim.y * bz);
    const unsigned logical = (linear % 8u) * (total / 8u) + linear / 8u;
    bx = logical % gridDim.x;
    by = (logical / gridDim.x) % gridDim.y;
    bz = logical / (gridDim.x * gridDim.y);
  }
  const int b = static_cast<int>(bz);
  const int chunk = static_cast<int>(bx) % P.max_chunks, rg = static_cast<int>(bx) / P.max_chunks;
  const int q0 = P.q_offsets[b];
  int n = P.q_offsets[b + 1] - q0;
  n = n > (WIDE ? kMaxQWide : kMaxQ) ? (WIDE ? kMaxQWide : kMaxQ) : n;
  const int ctx = P.ctx_len[b];
  const int L = ctx + n;
  const int nchunks = max(1, (L + P.chunk_tokens - 1) / P.chunk_tokens);
  const int cb = (((L + nchunks - 1) / nchunks) + RowsCfg<D, NW, SL>::kT - 1) & ~(RowsCfg<D, NW, SL>::kT - 1);
  rows_item<D, NW, WIDE, SL>(P, smem, b, static_cast<int>(by), chunk, rg, nchunks, cb, q0, n, ctx);
}

// Sorted-work-list launch for batches of up to kPlanMaxB requests with ragged lengths.  The grid
// is two workgroups per compute unit; every workgroup derives the same list of work items
// (request, chunk, KV head) from the lengths on the device, ordered by decreasing number of tiles
// a wave streams per item, and no workgroup is launched for chunks that do not exist.  A compute unit takes one item of the
// first 256 in order and one of the next 256 in reverse (its two workgroups), then two of each further 512: of a list that is
// short or steep at its head the shortest for the units that had the longest, else so that the sums of both workgroups stay even.
// Against rounds over the 512 workgroups, which gave a unit items i and 256 + i: 12 requests x 16 KV heads of 1000 to 7000
// tokens 110 -> 97 us, 32 x 8 122 -> 109, 128 x 8 of 512 to 6000 (steep) 179 -> 162; 32 x 32 of 1123 to 3922 is level (266 if
// taken for steep, 261).
// An item runs the token-split body or, for requests with many query rows, the row-split body.
template <int D>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_stream_list_kernel(AttnParams P) {
  using RC = RowsCfg<D, 4>;
  extern __shared__ __align__(256) unsigned char smem[];
  __shared__ int sh_first[kPlanMaxB + 1];        // first item of the request at sorted position s
  // the request at sorted position s: first query row (below 2^16) | nodes << 16 | request << 24, and its context
  // length: an item starts without a round trip to global memory for them
  __shared__ int sh_meta[kPlanMaxB], sh_ctx[kPlanMaxB];
  static_assert(kPlanMaxB <= 128 && kMaxQ <= 64, "request and node count share one word with the first query row");
  const int tid = threadIdx.x;
  int* key = reinterpret_cast<int*>(smem);       // scratch in the tile memory, dead before the first item
  int* cnt = key + kPlanMaxB;
  int my_key = -1, my_cnt = 0, my_meta = 0, my_ctx = 0;
  if (tid < P.B) {
    const int q0 = P.q_offsets[tid];
    int n = P.q_offsets[tid + 1] - q0;
    n = n > kMaxQ ? kMaxQ : (n < 0 ? 0 : n);
    const int ctx = P.ctx_len[tid];
    my_meta = q0 | (n << 16) | (tid << 24);
    my_ctx = ctx;
    if (n > 0) {
      const int L = ctx + n;
      const int nch = request_chunks(P, L, n);
      my_key = (request_units(P, L, n) + nch - 1) / nch;   // length of one item of this request
      my_cnt = nch * P.Hkv;
    }
  }
  if (tid < kPlanMaxB) { key[tid] = my_key; cnt[tid] = my_cnt; }
  __syncthreads();
  if (tid < P.B) {
    int rank = 0, first = 0;
    for (int j = 0; j < P.B; ++j) {
      const int kj = key[j];
      const bool before = kj > my_key || (kj == my_key && j < tid);
      rank += before ? 1 : 0;
      first += before ? cnt[j] : 0;
    }
    sh_meta[rank] = my_meta;
    sh_ctx[rank] = my_ctx;
    sh_first[rank] = first;
    if (rank == P.B - 1) sh_first[P.B] = first + my_cnt;
  }
  __syncthreads();
  const int total = sh_first[P.B];
  auto at_item = [&](int item) __attribute__((always_inline)) {     // sorted position of its request: largest s with sh_first[s] <= item
    int lo = 0, hi = P.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (sh_first[mid] <= item) lo = mid; else hi = mid;
    }
    return lo;
  };
  const int grid = static_cast<int>(gridDim.x), half = grid / 2, wg = static_cast<int>(blockIdx.x);
  const int unit = wg < half ? wg : wg - half;               // compute unit, with its two workgroups
  const int place = wg < half ? unit : grid - 1 - unit;
  bool skewed = true;             // the longest and the shortest of the first two turns together are well ahead of the two in the middle
  if (total > grid + half) {
    const int lane = tid & 63, at = lane == 0 ? 0 : (lane == 1 ? half - 1 : (lane == 2 ? half : grid - 1));
    const int s = at_item(at), n = (sh_meta[s] >> 16) & 0xff, L = sh_ctx[s] + n, nch = request_chunks(P, L, n);
    const int len = (request_units(P, L, n) + nch - 1) / nch;
    auto of = [&](int l) { return __builtin_amdgcn_readlane(len, l); };
    skewed = 10 * (of(0) + of(3)) > 11 * (of(1) + of(2));
  }
  for (int round = 0;; ++round) {
    int item = place;
    if (round > 0) item = skewed ? (wg < half ? half : grid) - 1 - unit : ((round & 1) ? grid - 1 - place : place);
    item += round * grid;
    if (round * grid >= total) break;
    if (item >= total) continue;
    const int lo = at_item(item);
    const int meta = sh_meta[lo];
    const int b = meta >> 24, q0 = meta & 0xffff, n = (meta >> 16) & 0xff, ctx = sh_ctx[lo];
    const int local = item - sh_first[lo];
    const int L = ctx + n;
    const int nch = request_chunks(P, L, n);
    const int cb = (((L + nch - 1) / nch) + RC::kT - 1) & ~(RC::kT - 1);
    // (a chunk longer than the row-split body's page table in LDS stays with the token-split body)
    if (list_uses_rows(P, n) && cb <= RC::kMaxChunkPages * kPage) rows_item<D, 4>(P, smem, b, local % P.Hkv, local / P.Hkv, 0, nch, cb, q0, n, ctx);
    else stream_item<D, kAttnWaves>(P, smem, b, local % P.Hkv, local / P.Hkv, 0, q0, n, ctx);
    __syncthreads();                              // the tile memory is reused by the next item
  }
}

// Grid-mapped launch of both bodies, for ragged batches with little work whose larger requests have 65 to 128 query rows
// per KV head: the body follows each request's own row count, as in the work list, so that a request of up to 64 rows
// keeps its two-term bf16 weights and its four waves whatever the largest request of the batch is.
template <int D>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_mixed_kernel(AttnParams P) {
  using RC = RowsCfg<D, 4>;
  extern __shared__ __align__(256) unsigned char smem[];
  const int b = P.chunks_last ? blockIdx.y : blockIdx.z, kvh = P.chunks_last ? blockIdx.x : blockIdx.y;
  const int chunk = P.chunks_last ? blockIdx.z : blockIdx.x;
  const int q0 = P.q_offsets[b];
  int n = P.q_offsets[b + 1] - q0;
  n = n > kMaxQ ? kMaxQ : n;
  const int ctx = P.ctx_len[b], L = ctx + n;
  const int nch = request_chunks(P, L, n);
  const int cb = (((L + nch - 1) / nch) + RC::kT - 1) & ~(RC::kT - 1);
  // (a chunk longer than the row-split body's page table in LDS stays with the token-split body)
  if (list_uses_rows(P, n) && cb <= RC::kMaxChunkPages * kPage) rows_item<D, 4>(P, smem, b, kvh, chunk, 0, nch, cb, q0, n, ctx);
  else stream_item<D, kAttnWaves>(P, smem, b, kvh, chunk, 0, q0, n, ctx);
}

// Merge the per-chunk partials of every (query row, head) that spans several chunks.  A group of D/4 lanes reads
// whole partial rows (16 bytes per lane) and S groups share one (node, head) row, group s taking chunks s, s + S, ...
// four at a time with their loads in flight together; the groups meet in LDS.  The kernel is bound by the latency of
// those loads, so S grows with the number of chunks (launch_combine): one request with 448 rows in 32 chunks took
// 20.7 us with one group per row walking the chunks one by one and takes 4.0 us with eight groups.
template <int D, int S>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnParams P) {
  constexpr int kLanes = D / 4;                 // lanes of a group
  constexpr int kGroups = 256 / kLanes;         // groups of a workgroup
  constexpr int kRows = kGroups / S;            // (node, head) rows of a workgroup
  constexpr int kFly = 4;                       // partial rows in flight per group
  // blockIdx.y = request
  const int b = blockIdx.y;
  const int q0 = P.q_offsets[b];
  int n = P.q_offsets[b + 1] - q0;
  n = n > P.n_cap ? P.n_cap : n;
  // both uniform over the workgroup; in large batches most workgroups leave here
  if (static_cast<int>(blockIdx.x) * kRows >= n * P.Hq) return;
  const int nchunks = request_chunks(P, P.ctx_len[b] + n, n);
  if (nchunks == 1) return;
  const int grp = threadIdx.x / kLanes, gl = threadIdx.x % kLanes;
  const int s = grp % S, local = blockIdx.x * kRows + grp / S;
  const bool ok = local < n * P.Hq;
  const int64_t grow = static_cast<int64_t>(q0) * P.Hq + (ok ? local : 0);
  const float2* ml = P.ws_ml + grow * P.max_chunks;
  const float* part = P.ws_o + grow * P.max_chunks * D + gl * 4;
  float M = -INFINITY, W = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int c0 = s; c0 < nchunks; c0 += S * kFly) {
    float2 st[kFly];
    float4 o[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int c = c0 + u * S;
      const int cc = c < nchunks ? c : c0;      // chunks past the end repeat the first of the batch, with weight 0
      st[u] = ml[cc];
      o[u] = *reinterpret_cast<const float4*>(part + static_cast<int64_t>(cc) * D);
      if (c >= nchunks) st[u].x = -INFINITY;
    }
    float m = M;
#pragma unroll
    for (int u = 0; u < kFly; ++u) m = fmaxf(m, st[u].x);
    const float mm = m == -INFINITY ? 0.f : m;
    const float a = fast_exp2(M - mm);
    W *= a; acc.x *= a; acc.y *= a; acc.z *= a; acc.w *= a;
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      if (st[u].x == -INFINITY) continue;       // a chunk without allowed positions (its partial row is not looked at)
      const float f = fast_exp2(st[u].x - mm);
      W += st[u].y * f;
      acc.x += o[u].x * f; acc.y += o[u].y * f; acc.z += o[u].z * f; acc.w += o[u].w * f;
    }
    M = m;
  }
  if constexpr (S > 1) {
    __shared__ float4 sh_acc[kGroups][kLanes];
    __shared__ float2 sh_ml[kGroups];
    sh_acc[grp][gl] = acc;
    if (gl == 0) sh_ml[grp] = make_float2(M, W);
    __syncthreads();
    if (s != 0) return;
    float m = M;
#pragma unroll
    for (int k = 1; k < S; ++k) m = fmaxf(m, sh_ml[grp + k].x);
    const float f0 = M == -INFINITY ? 0.f : fast_exp2(M - m);
    W *= f0; acc.x *= f0; acc.y *= f0; acc.z *= f0; acc.w *= f0;
#pragma unroll
    for (int k = 1; k < S; ++k) {
      const float2 t = sh_ml[grp + k];
      const float f = t.x == -INFINITY ? 0.f : fast_exp2(t.x - m);
      const float4 v = sh_acc[grp + k][gl];
      W += t.y * f;
      acc.x += v.x * f; acc.y += v.y * f; acc.z += v.z * f; acc.w += v.w * f;
    }
    M = m;
  }
  if (!ok) return;
  const float inv = 1.f / W;
  if (P.out_f32) {
    *reinterpret_cast<float4*>(static_cast<float*>(P.out) + grow * D + gl * 4) =
        make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  } else {
    uint2 o;
    o.x = pack_bf16(acc.x * inv, acc.y * inv);
    o.y = pack_bf16(acc.z * inv, acc.w * inv);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(P.out) + grow * D + gl * 4) = o;
  }
  if (P.lse && gl == 0) P.lse[grow] = (M + log2f(W)) * static_cast<float>(kLn2);
}

// ----------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------
constexpr int kListMaxChunks = 16;

// Development knobs for sweeps, compiled in only with -DSPECV_DEV_KNOBS (normal builds read no
// environment variable and keep no state between calls).
#ifdef SPECV_DEV_KNOBS
static long dev_knob(const char* name, long fallback) {
  const char* e = getenv(name);
  return e ? atol(e) : fallback;
}
#else
static long dev_knob(const char*, long fallback) { return fallback; }
#endif

// Longest item of the list in units.  An item longer than an average workgroup's share sets the end of the launch, a cut costs
// partial results and a merge.  At 36, 32, 30, 28 units: the serving mix (64 requests x 8 KV heads, 16 to 80 rows) 167, 168, 168,
// 168 us, 128 x 8 of 512 to 6000 tokens 167, 161, 162, 161, 16 x 8 of 4400 to 16000 117, 114, 114, 113, 12 x 16 of 4300 to 13600
// 190, 200, 201, 196, 32 x 32 of 512 to 16384 248, 251, 250, 261, of 1123 to 3922 (up to 31 units) 265, 265,
// 273, 276.
constexpr int kListTau = 32;
// ... where the items of kListTau units would be just more than one or two per compute unit and these are not (list_tau).
constexpr int kListTauFew[] = {40, 44};
// ... of an item that runs the row-split body: 38, 40, 42, 44, 46 units are 3891, 4096, 4301, 4506, 4710 tokens.  Averages over forty seeds
// of the serving mix 157.8, 157.5, 157.4, 158.2, 159.3 us, at worst 2, 2, 3, 11, 12 % behind the best of a seed; over 55 batches with
// more such requests (5 to 16 drafts each, or ten, twelve, sixteen; 32 or 64 requests) 44 is 0.8 % behind 42.
constexpr int kListTauRows = 42;
// Most chunks the work list cuts a request into: the longest one the block table can hold, in items of kListTau units for up
// to 32 rows.  More rows count twice and four times the waves they take, at 44: an upper bound, which sizes the workspace.
// least: ... for a workspace that does not hold that many, as one that was sized without a hint (chunks of up to 5120 tokens)
// may not: items of up to 44 units (5632 tokens).  The kernels lengthen the items of a request that is cut into more.
static int list_max_chunks(int64_t max_tok, int max_rows, bool least) {
  const int64_t tiles = (max_tok + kTile - 1) / kTile;
  const int64_t per_chunk = max_rows <= 32 ? (least ? 4 * 44 : 4 * kListTau) : (max_rows <= 64 ? 88 : 44);
  const int64_t mc = (tiles + per_chunk - 1) / per_chunk;
  return static_cast<int>(mc < 1 ? 1 : (mc > kListMaxChunks ? kListMaxChunks : mc));
}
// Units per item.  Batches of like lengths make pairs * (units of a request / units of an item + 1/2) items; when those spill over
// one or two per compute unit, some get one more than the others and the launch waits for them.  Of 164 batches of 48 to 256
// pairs (3000 to 16000 tokens, even and lognormal, 4 to 64 rows) the rule takes 40 units in 46: 9 % faster
// on average (6 x 16 of 4278 to 13606 tokens 115 -> 101 us, 24 x 8 of 4278 to 13606 190 -> 175), at worst 2 % slower (5 x 16 of 9000 to
// 16000: 97 -> 99); and 44 in 13: 4 % (3 x 32 of 9000 to 16000 128 -> 113), at worst 2 %.  At the line itself (18 batches of 256 to 262
// items estimated) both are even on average, 15 % faster to 7 % slower; below it (225 to 255) the shorter items are 2 % ahead.
// Items of 36 units ahead of these gain nothing; for a third item per compute unit the estimate is too rough (32 x 8 of 9000 to
// 16000: 319 -> 339).
static int list_tau(const AttnArgs& a, int64_t pairs, int max_rows) {
  if (max_rows > 64 || a.kv_hint <= 0) return kListTau;               // (a unit is 128 tokens for up to 64 rows)
  const double units = static_cast<double>(a.kv_hint) / a.B / (4 * kTile);
  auto items = [&](int tau) { return static_cast<double>(pairs) * (units / tau + 0.5); };
  const int n_cu = current_device_cus();
  for (int most = n_cu; most <= 2 * n_cu; most += n_cu)
    for (int tau : kListTauFew)
      if (items(kListTau) > most && items(tau) <= most) return tau;
  return kListTau;
}
// The launch for little work has a workgroup for every chunk a request could have.  Most chunks per request such that
// those are at most sixteen workgroups per compute unit, or two per (request, KV head) pair.
static int little_room(int64_t pairs) { return std::max<int>(2, static_cast<int>(4096 / std::max<int64_t>(pairs, 1))); }

AttnPlan make_attn_plan(const AttnArgs& a, bool small_workspace) {
  AttnPlan p;
  p.tau = 0;
  p.waves8 = 0;
  p.mixed = 0;
  p.wide_table = 0;
  p.wide = a.max_q > kMaxQ ? 1 : 0;
  const int G = a.Hq / a.Hkv;
  const int max_rows = a.max_q * G;
  const int64_t max_tok = static_cast<int64_t>(a.max_pages) * a.page;
  const bool ragged = a.kv_hint > 0 && a.kv_hint * 100 < static_cast<int64_t>(85) * a.B * max_tok;
  // Little work - the tokens of all requests and KV heads, dealt to 256 workgroups, are chunks below 1024 - is cut by
  // tokens, whatever the lengths: every request then has items of about one length.  The sorted work list cuts by what
  // a wave can stream at full load and left such batches to a few workgroups (5 requests x 4 KV heads, 777 to 3001
  // tokens: 20 of 512 workgroups, 26.7 us; 13.2 us cut into 512-token chunks).  The list serves them all the same where
  // a wide block table (allocated for the longest context a model allows) would ask for more chunks than there is room
  // for, and where the caller's workspace holds the list's partial results but not these (small_workspace).
  const int list_chunks = list_max_chunks(max_tok, max_rows, small_workspace);
  const int64_t pairs = static_cast<int64_t>(a.B) * a.Hkv;
  const int room = little_room(pairs);
  // Batches of up to 128 pairs of request and KV head go further (chunks below 1792), where the list has too few items for its
  // 512 workgroups: 4 requests x 16 KV heads of 1174 to 3487 tokens 43 -> 22 us, 8 x 4 of 6000 to 14600 65 -> 48, 6 x 16 of 1200 to
  // 5700 54 -> 40, 32 x 4 of 1000 to 7800 70 -> 66; at chunks above 2000 the list is even (8 x 8 of 6000 to 14600 78 and 81) or ahead.
  const int64_t little_tokens = static_cast<int64_t>(256) * (pairs <= 128 ? 1792 : 1024);
  const bool little = !small_workspace && a.kv_hint > 0 && a.kv_hint * a.Hkv < little_tokens && list_chunks <= room;
  // Up to 64 query rows per KV head the token-split body streams as fast as memory delivers; beyond, its
  // waves (one per 32-row block, each staging every tile for itself) are bound by their own staging and the
  // row-split body, whose waves share each staged tile, is ahead on batches of like lengths (96 rows per KV
  // head: 4.2 against 2.6 TB/s).  In ragged batches of up to 128 rows every request takes the body of its own row count
  // (work list, or attn_mixed_kernel when there is little work): max_q is a bound, and most requests have fewer nodes.
  if (max_rows <= 64 || (max_rows <= 128 && ragged && a.B <= kPlanMaxB)) { p.kind = 0; p.rows_per_wg = 128; }
  else if (max_rows <= 128 || a.D != 128) { p.kind = 1; p.rows_per_wg = 128; }
  else { p.kind = 2; p.rows_per_wg = 256; }
  // Few (request, KV head) pairs with many rows each: 256-row workgroups would have to cut the context to fill
  // the chip (partial results through memory and a combine kernel).  The sliced variant gives every pair twice
  // the workgroups instead - 128 rows each, the token halves of every tile split between two waves - when one
  // such workgroup per compute unit covers the batch.
  if (p.kind == 2) {
    const int64_t groups256 = static_cast<int64_t>(a.B) * a.Hkv * ((max_rows + 255) / 256);
    const int64_t groups128 = static_cast<int64_t>(a.B) * a.Hkv * ((max_rows + 127) / 128);
    const int n_cu = current_device_cus();
    if (groups256 * 4 <= 3 * static_cast<int64_t>(n_cu) && groups128 <= n_cu + n_cu / 4) { p.kind = 3; p.rows_per_wg = 128; }
  }
  const long force_kind = dev_knob("SPECV_ATTN_KIND", -1);            // force a kernel family
  if (force_kind == 1) { p.kind = 1; p.rows_per_wg = 128; }
  if (force_kind == 2 && a.D == 128) { p.kind = 2; p.rows_per_wg = 256; }
  if (force_kind == 0) { p.kind = 0; p.rows_per_wg = 128; }
  if (force_kind == 3 && a.D == 128 && max_rows > 128) { p.kind = 3; p.rows_per_wg = 128; }
  // more than 64 query nodes per request (two mask words per node): the row-split kernels only
  if (p.wide && p.kind == 0) { p.kind = 1; p.rows_per_wg = 128; }
  p.row_groups = (max_rows + p.rows_per_wg - 1) / p.rows_per_wg;
  // (the list kernel packs a request's first query row into 16 bits)
  const bool listable = p.kind == 0 && a.B <= kPlanMaxB && a.total_q < 65536;
  p.mixed = (listable && max_rows > 64 && little) ? 1 : 0;
  const bool token_split = (p.kind == 0 && !p.mixed);                           // (a mixed launch is cut for the row-split body)
  const int gran = token_split ? kTile : (p.kind == 3 ? 128 : 64);              // chunks are whole tiles
  int64_t tok = a.kv_hint > 0 ? a.kv_hint : static_cast<int64_t>(a.B) * max_tok;
  // Chunk length.  Every workgroup pays a fixed prologue/epilogue (and, when a request is split, a
  // partial-result round trip proportional to its query rows), so chunks are as long as two
  // limits allow: (a) about one workgroup per compute unit should exist, (b) a chunk of the token-split body should not
  // exceed 5120 tokens (40 tiles for each of four waves) for up to 32 rows, 2560 for up to 64, 1280 for more, or the longest
  // workgroup sets the kernel's duration.
  const long jobs_knob = dev_knob("SPECV_ATTN_JOBS", 0);
  const int64_t jobs_target = jobs_knob > 0 ? jobs_knob : (p.kind == 1 || p.mixed ? 512 : 256);   // 4-wave row-split body: two per compute unit
  int64_t chunk = (tok * a.Hkv * p.row_groups + jobs_target - 1) / jobs_target;
  if (token_split && jobs_knob <= 0) {
    const int64_t cap = max_rows <= 32 ? 5120 : (max_rows <= 64 ? 2560 : 1280);
    if (chunk > cap) chunk = cap;
  }
  // shortest chunk: two tiles per wave of the eight-wave token-split kernel (which such launches take, below); a shorter
  // one saves a wave one tile and costs every request a merge (1 request of 260 tokens: one launch instead of two)
  const int64_t shortest = token_split ? 512 : 256;
  if (chunk < shortest) chunk = shortest;
  // Ragged batches with little work, but with a workgroup for half of the compute units before any cut, stay whole where
  // the longest request is at most 1536 tokens (up to 32 rows), 768 (up to 64) or 1008 long: a cut saves the longest workgroups less
  // time than the partial results and a merge launch over all query rows take.  Whole against cut: 100
  // requests x 8 KV heads of 20 to 500 tokens (up to 120 rows) 36.9 and 57.6 us (list 39.2), 20 x 32 of 20 to 500 28.8 and
  // 49.0 (30.6), 40 x 8 of 20 to 700 (up to 32 rows) 20.8 and 28.5 (23.2), 25 x 8 of 20 to 500 18.8 and 20.5 (22.6); with 25 x
  // 8 of 100 to 500 and three of 4000 tokens cutting stays ahead, 24.7 against 33.2.
  if (little && ragged && p.kind == 0 && pairs >= 128 &&
      max_tok <= (max_rows <= 32 ? 1536 : (max_rows <= 64 ? 768 : 1008)))
    chunk = std::max(chunk, max_tok);
  chunk = (chunk + gran - 1) / gran * gran;
  if (chunk > max_tok) chunk = (max_tok + gran - 1) / gran * gran;
  // the row-split kernel keeps a chunk's page ids in LDS
  const int64_t rows_chunk_cap = (p.kind >= 2) ? 16384 : 8192;
  if (!token_split && chunk > rows_chunk_cap) chunk = rows_chunk_cap;
  if (chunk < gran) chunk = gran;
  p.chunk_tokens = static_cast<int>(chunk);
  p.max_chunks = static_cast<int>((max_tok + chunk - 1) / chunk);
  if (p.max_chunks < 1) p.max_chunks = 1;
  // Small batches whose lengths are ragged run the token-split kernel from a sorted work list built
  // on the device (the lengths are device data); there chunks are cut by tiles per wave, not by
  // tokens.  The list costs every workgroup one extra round of dependent loads (~5 us per launch),
  // which only pays when lengths differ: the caller's total-token hint against batch x longest
  // request says whether they do.
  int tau = (listable && ragged && !little) ? list_tau(a, pairs, max_rows) : 0;
  const long tau_knob = dev_knob("SPECV_ATTN_TAU", -1);   // 0: grid-mapped launch
  if (listable && !p.mixed && tau_knob >= 0 && tau_knob <= 255) tau = static_cast<int>(tau_knob);
  if (jobs_knob > 0) tau = 0;
  if (tau > 0) {
    p.tau = tau;
    p.max_chunks = list_chunks;
  } else if (listable && ragged) {
    // A table much wider than the requests - it would launch four times the workgroups that the hint's tokens and one
    // partial chunk per request make, or it is wider than all tokens together are long: the workgroups without a chunk go
    // last (chunks_last), and there are no more chunks than the list would make, eight, or twice those of an average
    // request (one request: its own); a request that is longer than so many is cut into longer ones.  Launch, partial
    // results and the groups that merge them follow the tokens, not the table.
    const int64_t all = (tok + p.chunk_tokens - 1) / p.chunk_tokens, launched = p.max_chunks * pairs;
    if ((launched > 1024 && launched > 4 * (all * a.Hkv + pairs)) || p.max_chunks > all + 1) {
      int64_t bound = a.B > 1 ? 2 * all / a.B : all;
      bound = std::min<int64_t>(std::max<int64_t>(bound, std::max(list_chunks, 8)), room);
      p.max_chunks = static_cast<int>(std::min<int64_t>(bound, p.max_chunks));
      p.wide_table = 1;
    }
  }
  if (token_split && p.tau == 0) {
    // one workgroup of eight waves per compute unit where there are not two of four for it; workgroups that have work:
    // at most what the hint's tokens and one partial chunk per request make
    const int64_t jobs = (tok / p.chunk_tokens + a.B) * a.Hkv * p.row_groups;
    const int64_t most = static_cast<int64_t>(p.max_chunks) * a.B * a.Hkv * p.row_groups;
    p.waves8 = (jobs < most ? jobs : most) <= current_device_cus() ? 1 : 0;
  }
  return p;
}

size_t attn_workspace_bytes(const AttnArgs& a, const AttnPlan& p) {
  if (p.max_chunks <= 1) return 256;
  const size_t rows = static_cast<size_t>(a.total_q) * a.Hq;
  return rows * p.max_chunks * (a.D + 2) * sizeof(float) + 256;
}

const char* attn_plan_name(const AttnPlan& p) {
  if (p.mixed) return "attn_mixed_kernel (one workgroup per request x KV head x context chunk; token-split body, row-split body from 65 query rows per KV head)";
  if (p.kind == 0) return p.tau > 0 ? "attn_stream_list_kernel (device-built work list sorted by length; token-split body, row-split body from 65 query rows per KV head)"
                                    : "attn_stream_kernel (token-split body, one workgroup per request x KV head x context chunk)";
  if (p.kind == 1) return "attn_rows_kernel<4 waves> (row-split body)";
  if (p.kind == 3) return "attn_rows_kernel<8 waves, sliced> (row-split body, 128 query rows per workgroup, two waves per 32-row block)";
  return "attn_rows_kernel<8 waves> (row-split body, 256 query rows per workgroup)";
}

// token-split body: a tile of K and one of V per wave, a query block, masks and parents; the merge takes the same memory
template <int D>
constexpr size_t stream_lds(int NW) {
  return std::max(2 * static_cast<size_t>(NW) * AttnCfg<D>::kTileBytes + AttnCfg<D>::kQLdsFrags * 1024 + kMaxQ * 12,
                  static_cast<size_t>(NW) * 32 * (AttnCfg<D>::kORedStride + 2) * sizeof(float));
}

// kernels with both four-wave bodies: the tile memory of the larger one
template <int D>
constexpr size_t both_bodies_lds() {
  return std::max(stream_lds<D>(kAttnWaves), static_cast<size_t>(RowsCfg<D, 4>::kLds));
}

template <int D>
static int launch_stream_list(const AttnParams& P, hipStream_t stream) {
  constexpr size_t kListLds = both_bodies_lds<D>();
  // two workgroups per compute unit: dynamic plus the kernel's static LDS (1792 bytes with its alignment) within half of 160 KB
  static_assert(kListLds + 1792 <= 80 * 1024, "the work-list kernel must fit twice into a compute unit's LDS");
  static std::atomic<uint64_t> list_attr_done{0};
  if (set_lds_once(&attn_stream_list_kernel<D>, kListLds, list_attr_done) != 0) return -6;
  const int n_cu = current_device_cus();
  hipLaunchKernelGGL((attn_stream_list_kernel<D>), dim3(2 * n_cu), dim3(kAttnThreads), kListLds, stream, P);
  return hipGetLastError() == hipSuccess ? 0 : -6;
}

static dim3 stream_grid(const AttnParams& P, const AttnPlan& plan, int B, int Hkv) {
  const int cuts = plan.max_chunks * plan.row_groups;
  return P.chunks_last ? dim3(Hkv, B, cuts) : dim3(cuts, Hkv, B);
}

template <int D>
static int launch_mixed(const AttnParams& P, const AttnPlan& plan, int B, int Hkv, hipStream_t stream) {
  constexpr size_t kLds = both_bodies_lds<D>();
  static_assert(kLds <= 80 * 1024, "two workgroups of the mixed kernel per compute unit");
  static std::atomic<uint64_t> attr_done{0};
  if (set_lds_once(&attn_mixed_kernel<D>, kLds, attr_done) != 0) return -6;
  hipLaunchKernelGGL((attn_mixed_kernel<D>), stream_grid(P, plan, B, Hkv), dim3(kAttnThreads), kLds, stream, P);
  return hipGetLastError() == hipSuccess ? 0 : -6;
}

template <int D, int NW>
static int launch_stream_as(const AttnParams& P, const AttnPlan& plan, int B, int Hkv, hipStream_t stream) {
  constexpr size_t kTiles = stream_lds<D>(NW);
  static_assert(kTiles * (NW == 4 ? 2 : 1) <= 160 * 1024, "token-split kernel: LDS per compute unit");
  static std::atomic<uint64_t> attr_done{0};
  if (set_lds_once(&attn_stream_kernel<D, NW>, kTiles, attr_done) != 0) return -6;
  hipLaunchKernelGGL((attn_stream_kernel<D, NW>), stream_grid(P, plan, B, Hkv), dim3(NW * kWave), kTiles, stream, P);
  return hipGetLastError() == hipSuccess ? 0 : -6;
}

template <int D>
static int launch_stream(const AttnParams& P, const AttnPlan& plan, int B, int Hkv, hipStream_t stream) {
  if (plan.tau > 0) return launch_stream_list<D>(P, stream);
  if (plan.mixed) return launch_mixed<D>(P, plan, B, Hkv, stream);
  return plan.waves8 ? launch_stream_as<D, 8>(P, plan, B, Hkv, stream) : launch_stream_as<D, 4>(P, plan, B, Hkv, stream);
}

template <int D, int NW, bool WIDE, int SL = 1>
static int launch_rows_as(const AttnParams& P, const AttnPlan& plan, int B, int Hkv, hipStream_t stream) {
  using RC = RowsCfg<D, NW, SL>;
  constexpr size_t kLds = RC::lds_bytes(WIDE);
  static_assert(kLds * (NW == 4 ? 2 : 1) <= 160 * 1024, "row-split kernel: LDS per compute unit");
  static std::atomic<uint64_t> attr_done{0};
  if (set_lds_once(&attn_rows_kernel<D, NW, WIDE, SL>, kLds, attr_done) != 0) return -6;
  dim3 grid(plan.max_chunks * plan.row_groups, Hkv, B);
  hipLaunchKernelGGL((attn_rows_kernel<D, NW, WIDE, SL>), grid, dim3(RC::kThreads), kLds, stream, P);
  return hipGetLastError() == hipSuccess ? 0 : -6;
}

template <int D, int NW>
static int launch_rows(const AttnParams& P, const AttnPlan& plan, int B, int Hkv, hipStream_t stream) {
  return plan.wide ? launch_rows_as<D, NW, true>(P, plan, B, Hkv, stream) : launch_rows_as<D, NW, false>(P, plan, B, Hkv, stream);
}

template <int D, int S>
static int launch_combine_as(const AttnArgs& a, const AttnParams& P, hipStream_t stream) {
  constexpr int kRows = 256 / (D / 4) / S;
  const int max_q = a.max_q > P.n_cap ? P.n_cap : a.max_q;
  hipLaunchKernelGGL((attn_combine_kernel<D, S>), dim3((max_q * a.Hq + kRows - 1) / kRows, a.B), dim3(256), 0, stream, P);
  return hipGetLastError() == hipSuccess ? 0 : -6;
}

// Groups of lanes per merged row: a group keeps four partial rows in flight, so four chunks per group are one round
// trip to memory and more groups than that only cost workgroups.  Large launches have enough rows to fill the chip:
// there the groups would multiply workgroups most of which find a request that was not cut.
template <int D>
static int launch_combine(const AttnArgs& a, const AttnParams& P, const AttnPlan& plan, hipStream_t stream) {
  constexpr int kGroups = 256 / (D / 4);
  const int max_q = a.max_q > P.n_cap ? P.n_cap : a.max_q;
  const int64_t rows = static_cast<int64_t>(max_q) * a.Hq * a.B;
  int S = 1;
  while (S < 8 && 4 * S < plan.max_chunks && rows * 2 * S <= static_cast<int64_t>(kGroups) * 2048) S *= 2;
  if (S == 1) return launch_combine_as<D, 1>(a, P, stream);
  if (S == 2) return launch_combine_as<D, 2>(a, P, stream);
  if (S == 4) return launch_combine_as<D, 4>(a, P, stream);
  return launch_combine_as<D, 8>(a, P, stream);
}

int launch_attn(const AttnArgs& a, const AttnPlan& plan, hipStream_t stream) {
  if (a.B <= 0 || a.total_q <= 0) return 0;
  AttnParams P;
  P.q = static_cast<const uint16_t*>(a.q);
  P.k_pool = static_cast<const uint16_t*>(a.k_pool);
  P.v_pool = static_cast<const uint16_t*>(a.v_pool);
  P.block_table = a.block_table; P.ctx_len = a.ctx_len; P.q_offsets = a.q_offsets; P.parent = a.parent;
  P.out = a.out; P.lse = a.lse;
  const size_t rows = static_cast<size_t>(a.total_q) * a.Hq;
  P.ws_ml = static_cast<float2*>(a.workspace);
  P.ws_o = reinterpret_cast<float*>(static_cast<unsigned char*>(a.workspace) +
                                    ((rows * plan.max_chunks * sizeof(float2) + 255) / 256) * 256);
  P.B = a.B; P.Hq = a.Hq; P.Hkv = a.Hkv; P.G = a.Hq / a.Hkv; P.max_pages = a.max_pages;
  P.chunk_tokens = plan.chunk_tokens; P.max_chunks = plan.max_chunks; P.tau = plan.tau;
  // both bodies: from 65 query rows per KV head (three 32-row blocks) on, a request runs the row-split body
  P.list_rows_min = plan.tau > 0 || plan.mixed ? static_cast<int>(dev_knob("SPECV_ATTN_LIST_ROWS", 65)) : 0;
  P.tau_rows = static_cast<int>(dev_knob("SPECV_ATTN_TAU_ROWS", kListTauRows));
  P.list_rows_units = static_cast<int>(dev_knob("SPECV_ATTN_ROWS_UNITS", 5));
  P.n_cap = plan.wide ? kMaxQWide : kMaxQ;
  P.chunks_last = plan.wide_table;
  P.xcd_swizzle = (plan.kind != 0 && plan.row_groups > 1 &&
                   (static_cast<int64_t>(plan.max_chunks) * plan.row_groups * a.Hkv * a.B) % 8 == 0) ? 1 : 0;
  P.c = a.scale * kLog2e;
  P.out_f32 = (a.out_dtype == kF32);
  int rc;
  if (plan.kind == 0) rc = a.D == 128 ? launch_stream<128>(P, plan, a.B, a.Hkv, stream) : launch_stream<64>(P, plan, a.B, a.Hkv, stream);
  else if (plan.kind == 1) rc = a.D == 128 ? launch_rows<128, 4>(P, plan, a.B, a.Hkv, stream) : launch_rows<64, 4>(P, plan, a.B, a.Hkv, stream);
  else if (plan.kind == 2) rc = launch_rows<128, 8>(P, plan, a.B, a.Hkv, stream);
  else rc = plan.wide ? launch_rows_as<128, 8, true, 2>(P, plan, a.B, a.Hkv, stream)
                      : launch_rows_as<128, 8, false, 2>(P, plan, a.B, a.Hkv, stream);
  if (rc != 0) return rc;
  if (plan.max_chunks > 1) return a.D == 128 ? launch_combine<128>(a, P, plan, stream) : launch_combine<64>(a, P, plan, stream);
  return 0;
}

}  // namespace specv
