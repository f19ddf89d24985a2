// Acceptance-rejection walk of Section 2.1 (accept x when q(x) <= o(x), else reject with
// probability 1 - o(x)/q(x); replacement from norm(max(0, o - q)); bonus token when nothing is
// rejected; siblings of a draft tree by recursive rejection) for bf16 logit rows, as ONE kernel
// that reads only the rows the walk reaches.
//
// A request is walked by a cluster of C = LV x SL workgroups on different compute units.  The walk
// proceeds in windows: the current node and its chain of first children (LV levels, the speculated
// continuation of the walk).  Workgroup (lv, sl) loads vocabulary slice sl of the row pair of level
// lv (the node's target row and the draft row its children were drawn from) ONCE into its LDS,
// reduces its part of the softmax statistics, and all workgroups exchange their parts through small
// tagged messages in device memory.  Every workgroup then takes the same accept decisions from the
// same numbers (a replicated state machine: nothing has to be broadcast).  A rejection needs the
// mass of max(0, r - q): the workgroups of that level sum their slices (from registers or LDS) and exchange
// again; the final inverse-CDF draw locates the slice from the exchanged sums and the workgroup that
// holds it finds the token there.  The rows of the child under test are fetched before it is accepted; else rows
// behind the first rejection are never read.
//
// Messages.  One message = four 64-bit words {27 bits of data : 37-bit tag}, written with relaxed device-scope stores
// and read with relaxed device-scope loads; a word is valid when its tag is the call's plus the round number, so
// no ordering between words is needed.  Every workgroup posts in every round (a dummy when it has
// nothing to add) into one of two buffers chosen by the round's parity: a workgroup can post round
// r+2 only after it has seen every peer's round r+1, i.e. after every peer has finished reading
// round r, so two buffers suffice.  Whatever the buffers hold carries other tags (see next_message_tag), so nothing clears
// them (a kernel ahead that did cost 5 of 128 us of a step of 16 x 64 tree nodes), but for launches that are being
// captured: replays repeat their tag.  (37 bits of tag instead of 32, so that it does not come round: 0.4 us of 126; a fourth word
// to look at: 2 us.)
//
// No wait is unbounded and the result never depends on a peer making progress: a workgroup that does
// not see a round complete within its patience leaves; if it is the cluster's first workgroup (the
// owner, which writes the outputs) it marks its messages "abort" so the others leave too, and walks
// the request alone, computing every slice's part itself in the same order and with the same
// arithmetic (the results are bit-identical to the cluster's).  Clusters of one workgroup (large
// batches) work this way from the start.
#include "common.h"
#include "kernels.h"

namespace specv {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kClThreads = 256;             // four waves, one per SIMD: the per-wave reductions and the replicated
                                            // scalar steps cost a quarter of what sixteen waves would pay
constexpr int kClWaves = kClThreads / kWave;
// One more wave waits for the messages: loads return in order, and a wave with rows on their way would not see a message
// before them.  It takes part in the barriers and in the replicated state, and holds no logits.
constexpr int kClBlock = kClThreads + kWave;
constexpr int kClUnit = kClThreads * 8;        // logits one workgroup-wide 16-byte load covers (2048)
constexpr int kClNodes = 128;
constexpr int kClMaxUpt = 16;                  // units per slice: 16 x 4 KiB per row, two rows = 128 KiB of LDS
constexpr int kClMaxParts = kClMaxUpt * kClWaves;
constexpr unsigned kClAbort = kTagRounds - 1;  // added to the call's tag in place of a round number
constexpr uint32_t kNegInf2 = 0xff80ff80u;     // two bf16 -inf

// Words of a message that count: the maxima are of bf16 logits (one of them).
constexpr int kClWords = record_words(kBF16);

struct ClusterParams {
  int B, V, n_q_rows;
  const int32_t* node_offsets;
  const int32_t* parent;
  const int32_t* draft_tokens;
  const uint16_t* target;
  const uint16_t* draft_q;
  const int32_t* q_row;
  float c;                        // log2(e) / T
  const float* u_accept;
  const float* u_resample;
  int32_t* accept_len;
  int32_t* out_tokens; int out_stride;
  int32_t* stop_node;
  float* dbg_ratio;
  int LV, SL;                     // window levels x vocabulary slices = workgroups per request
  int UPT;                        // units (2048 logits) per slice
  int solo;                       // one workgroup per request, which computes all LV x SL parts itself
  unsigned long long tag;         // of the call's messages, plus the round number
  int patience;                   // polls the owner spends on one round before it walks alone
  unsigned long long* msg;        // [B][2 buffers][C][2 messages][4 words]
};

// 16 bytes per lane from base + off to LDS: lane i's land at byte lds_at + 16 i.  Not tracked by the compiler (the reader
// waits); the LDS address is an operand bound to M0.
__device__ __forceinline__ void cl_load_to_lds(const uint16_t* base, unsigned off, unsigned lds_at) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "{m0}"(lds_at), "v"(off), "s"(base) : "memory");
}

__device__ __forceinline__ void cl_unpack(u32x4 r, float (&x)[8]) {
  x[0] = bf16_lo(r[0]); x[1] = bf16_hi(r[0]); x[2] = bf16_lo(r[1]); x[3] = bf16_hi(r[1]);
  x[4] = bf16_lo(r[2]); x[5] = bf16_hi(r[2]); x[6] = bf16_lo(r[3]); x[7] = bf16_hi(r[3]);
}

// Statistics of one level of the window: row maxima and reciprocal sums of 2^((l - max) c).
struct LevelStats {
  float mp, mq;
  double izp, izq;
};

// Weights of eight consecutive classes at residual level L:
//   r_0 = p;  w_k = max(0, r_{k-1} - q);  r_k = w_k / R_k,  R_k = sum_v w_k(v);
// the weight of level L is w_L (unnormalised; p itself at level 0).  Classes beyond the vocabulary
// hold -inf logits and get weight 0.  Per-class values are fp32, sums over classes fp64.
__device__ __forceinline__ void cl_weights(u32x4 rp, u32x4 rq, const LevelStats& S, float c, int L,
                                           const float* __restrict__ inv_R, float (&w)[8]) {
  float lp[8], lq[8], q[8];
  cl_unpack(rp, lp);
  cl_unpack(rq, lq);
  const float izp = static_cast<float>(S.izp), izq = static_cast<float>(S.izq);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    w[j] = fast_exp2((lp[j] - S.mp) * c) * izp;
    q[j] = 0.f;
    if (L > 0) q[j] = fast_exp2((lq[j] - S.mq) * c) * izq;
  }
  for (int k = 0; k < L; ++k) {
    const float scale = (k + 1 < L) ? inv_R[k] : 1.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = fmaxf(w[j] - q[j], 0.f) * scale;
  }
}

// Barrier for what the waves of a workgroup exchange through LDS: rows on their way to LDS and stores to memory stay in flight.
__device__ __forceinline__ void cl_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// 2^x: 2^n by ldexp, 2^f for |f| <= 1/2 by the exponential series, 1 + f (ln 2 + f (...)) with the terms (f ln 2)^k / k! up to k = 13
// (the first one left out is 3e-18), even and odd powers side by side: the walk is a chain of such values.  The low bits of
// ln 2 go in with the small terms.  Largest error over [-60, 0] 0.86 of a last place (1.34e-16 relative, rms 4.8e-17), against
// 0.86 (1.36e-16, 4.9e-17) of the library's function.
__device__ __forceinline__ double cl_exp2(double x) {
  const double y = x < -2000.0 ? -2000.0 : x;             // (-inf: 0; NaN stays)
  const double n = __builtin_rint(y), f = y - n, g = f * f;
  auto k = [](double c) __attribute__((always_inline)) {  // (a scalar where it is used: kept in vector registers they fill 26 of them)
    asm volatile("" : "+s"(c));
    return c;
  };
  double even = fma(k(2.5678435993488206e-11), g, k(7.054911620801123e-09)), odd = fma(k(1.3691488853904128e-12), g, k(4.4455382718708116e-10));
  even = fma(even, g, k(1.321548679014431e-06)); odd = fma(odd, g, k(1.01780860092397e-07));
  even = fma(even, g, k(0.0001540353039338161)); odd = fma(odd, g, k(1.5252733804059841e-05));
  even = fma(even, g, k(0.009618129107628477)); odd = fma(odd, g, k(0.0013333558146428443));
  even = fma(even, g, k(0.24022650695910072)); odd = fma(odd, g, k(0.05550410866482158));
  const double rest = fma(f, fma(f, odd, even), k(2.3190468138462996e-17));
  return __builtin_ldexp(fma(f, k(0.6931471805599453) + rest, 1.0), static_cast<int>(n));
}

// Two wave reductions side by side (each step of one fills the waits of the other).
__device__ __forceinline__ void cl_max2(float& a, float& b) {
  a = dpp_max_step<0x111, 0xf>(a); b = dpp_max_step<0x111, 0xf>(b);
  a = dpp_max_step<0x112, 0xf>(a); b = dpp_max_step<0x112, 0xf>(b);
  a = dpp_max_step<0x114, 0xf>(a); b = dpp_max_step<0x114, 0xf>(b);
  a = dpp_max_step<0x118, 0xf>(a); b = dpp_max_step<0x118, 0xf>(b);
  a = dpp_max_step<0x142, 0xa>(a); b = dpp_max_step<0x142, 0xa>(b);
  a = dpp_max_step<0x143, 0xc>(a); b = dpp_max_step<0x143, 0xc>(b);
  a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 63));
  b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 63));
}
__device__ __forceinline__ void cl_sum2(double& a, double& b) {
  a += dpp_f64<0x111, 0xf>(a); b += dpp_f64<0x111, 0xf>(b);
  a += dpp_f64<0x112, 0xf>(a); b += dpp_f64<0x112, 0xf>(b);
  a += dpp_f64<0x114, 0xf>(a); b += dpp_f64<0x114, 0xf>(b);
  a += dpp_f64<0x118, 0xf>(a); b += dpp_f64<0x118, 0xf>(b);
  a += dpp_f64<0x142, 0xa>(a); b += dpp_f64<0x142, 0xa>(b);
  a += dpp_f64<0x143, 0xc>(a); b += dpp_f64<0x143, 0xc>(b);
  a = lane_f64(a, 63);
  b = lane_f64(b, 63);
}

// U: units per slice of a cluster whose slice is worked out once and kept in registers (4, the library's choice wherever
// every 8192-logit slice has a compute unit of its own): the exponentials that the statistics need are the weights up to a
// factor per row, so a rejection costs a subtraction per class instead of two exponentials, and the rows of the node under
// test are fetched into the LDS space that the raw slice has left.  U = 0: any number of units, read from LDS each time.
// What bounds it is a chain: per accepted node one exchange (1.2 us), the exponentials of the slice (0.7 us on its compute unit),
// reductions and fp64 scalars, per rejection one exchange.  16 trees of 64 nodes, 128256 classes: 52.6 -> 46.0 us (kernel) with
// weights kept, rows fetched ahead, the messages in a wave of their own (no barrier waits for a store or a row) and the scalar
// steps shortened; the same without that wave was 57.
template <int U>
__global__ __launch_bounds__(kClBlock) void accept_cluster_kernel(ClusterParams P) {
  // the slice this workgroup holds (or the one on its way): [target row, draft row][UPT units][thread] x 16 bytes; a thread
  // only ever touches its own 16-byte slots, so no barrier orders these accesses
  extern __shared__ __align__(16) unsigned char cl_rows[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int SL = P.SL, LV = P.LV, C = SL * LV, UPT = U ? U : P.UPT;
  const int CP = P.solo ? 1 : C;                  // workgroups that really exist per request
  const int b = blockIdx.x / CP, rank = blockIdx.x - b * CP;
  const int my_lv = rank / SL, my_sl = rank - my_lv * SL;
  const bool owner = rank == 0;
  const bool data = wave < kClWaves;              // this wave holds a part of the slice
  const int V = P.V;
  const float c = P.c;

  __shared__ int sh_par[kClNodes], sh_tok[kClNodes], sh_qrow[kClNodes];
  __shared__ float sh_u[kClNodes], sh_lp[kClNodes], sh_lq[kClNodes];   // uniforms; raw logits of the drafted tokens
  __shared__ int sh_fc[kClNodes + 1];          // first child of node cur at [cur + 1], -2 = none
  __shared__ int sh_out[kClNodes + 1];         // accepted tokens
  __shared__ double sh_val[64];                // gathered messages
  __shared__ float sh_aux[64];
  __shared__ float sh_M[2][16];                // per level: maximum of the target row / the draft row
  __shared__ double sh_iZ[2][16];              //            reciprocal sums
  __shared__ __align__(16) float sh_wm[2][kClWaves];
  __shared__ double sh_ws[2][kClWaves];        // per-wave sums of the slice held in LDS
  __shared__ double sh_part[kClMaxParts];      // its per-(unit, wave) sums (computed for the draw only)
  __shared__ double sh_invR[kClNodes];
  __shared__ float sh_invRf[kClNodes];
  __shared__ int sh_status;
  const int n_parts = UPT * kClWaves;          // <= 64

  const int o = P.node_offsets[b];
  int n = P.node_offsets[b + 1] - o;
  n = n < 0 ? 0 : (n > kClNodes ? kClNodes : n);
  const int64_t trow0 = static_cast<int64_t>(o) + b;
  const double u_res = static_cast<double>(P.u_resample[b]);

  // ---- slices: thread t holds chunk t of every unit.  They go from memory straight to LDS. ----
  auto row_p = [&](int u) -> u32x4* { return reinterpret_cast<u32x4*>(cl_rows) + (u * kClThreads + tid); };
  auto row_q = [&](int u) -> u32x4* { return reinterpret_cast<u32x4*>(cl_rows) + ((UPT + u) * kClThreads + tid); };
  const unsigned rows_at = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)cl_rows)) +
                           wave * kWave * 16;
  auto issue_rows = [&](const uint16_t* tp, const uint16_t* qp, int sl) {       // (qp may be null: no child)
    if (!data) return;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slots have been read
    int t = tid;
    asm volatile("" : "+v"(t));                            // (offsets are worked out here, see msg_at)
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      const int e = (sl * UPT + u) * kClUnit + t * 8;
      const unsigned off = e < V ? 2u * e : 0u;   // (V is a multiple of 8; chunks past the end are overwritten in settle)
      cl_load_to_lds(tp, off, rows_at + u * kClThreads * 16);
      if (qp) cl_load_to_lds(qp, off, rows_at + (UPT + u) * kClThreads * 16);
    }
  };
  auto settle = [&](bool child, int sl) {         // the rows are here
    if (!data) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const u32x4 ninf = {kNegInf2, kNegInf2, kNegInf2, kNegInf2};
    for (int u = 0; u < UPT; ++u) {
      const bool out = (sl * UPT + u) * kClUnit + tid * 8 >= V;
      if (out) *row_p(u) = ninf;
      if (out || !child) *row_q(u) = ninf;
    }
  };
  // the rows of this workgroup's level, when they are known before the node arrays arrive (the root's, whose first child is
  // node 0; any level of a linear draft): their loads go out first and overlap the dependent reads below
  const bool early = !P.solo && (my_lv == 0 || P.parent == nullptr) && my_lv - 1 < n;
  if (early) {
    const int qr = my_lv < n ? min(max(P.q_row[o + my_lv], 0), P.n_q_rows - 1) : 0;
    issue_rows(P.target + (trow0 + my_lv) * static_cast<int64_t>(V),
               my_lv < n ? P.draft_q + static_cast<int64_t>(__builtin_amdgcn_readfirstlane(qr)) * V : nullptr, my_sl);
  }

  // ---- node arrays, by the wave that holds no logits: its loads do not queue behind the rows.  (Indices come from device
  // memory the host cannot check: clamp them.)  Lane l takes nodes l and l + 64; the steps are ordered within the wave. ----
  int my_tok[2] = {0, 0}, my_prt[2] = {-1, -1};
  if (!data) {
    int qr[2] = {0, 0};
    float u[2] = {0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nd = lane + 64 * h;
      my_prt[h] = -2;
      if (nd < n) {
        my_prt[h] = P.parent ? P.parent[o + nd] : nd - 1;
        my_tok[h] = P.draft_tokens[o + nd];
        qr[h] = P.q_row[o + nd];
        u[h] = P.u_accept[o + nd];
        if (owner && P.dbg_ratio) P.dbg_ratio[o + nd] = __builtin_nanf("");
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nd = lane + 64 * h;
      if (nd < n && (my_prt[h] < -1 || my_prt[h] >= nd)) my_prt[h] = -1;
      my_tok[h] = min(max(my_tok[h], 0), V - 1);
      sh_par[nd] = my_prt[h]; sh_tok[nd] = my_tok[h]; sh_qrow[nd] = min(max(qr[h], 0), P.n_q_rows - 1); sh_u[nd] = u[h];
      sh_fc[nd] = kClNodes;
      sh_invRf[nd] = 0.f;
      sh_invR[nd] = 0.0;
    }
    if (lane == 0) sh_fc[kClNodes] = kClNodes;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (lane + 64 * h < n) atomicMin(&sh_fc[my_prt[h] + 1], lane + 64 * h);    // first child = lowest index among the children
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    for (int i = lane; i <= kClNodes; i += kWave)
      if (sh_fc[i] >= kClNodes) sh_fc[i] = -2;    // no child
  }
  cl_sync();
  // The two logits of every drafted token; the draft row of a sibling group is the one its first child names (the row the
  // slices hold for that group).  Read after the first exchange, whose barriers order it.
  if (!data) {
    float lp[2] = {0.f, 0.f}, lq[2] = {0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (lane + 64 * h < n) {
        const int fc = min(max(sh_fc[my_prt[h] + 1], 0), kClNodes - 1);
        lp[h] = bf16_bits_to_float(P.target[(trow0 + 1 + my_prt[h]) * static_cast<int64_t>(V) + my_tok[h]]);
        lq[h] = bf16_bits_to_float(P.draft_q[static_cast<int64_t>(sh_qrow[fc]) * V + my_tok[h]]);
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) { sh_lp[lane + 64 * h] = lp[h]; sh_lq[lane + 64 * h] = lq[h]; }
  }
  // lane l looks after nodes l and l + 64; nodes that do not exist hold an impossible parent
  const int my_parent = (lane < n) ? sh_par[lane] : -3;
  const int my_parent_hi = (lane + 64 < n) ? sh_par[lane + 64] : -3;

  auto issue_node = [&](int node, int sl) {         // node >= -1
    node = __builtin_amdgcn_readfirstlane(node);
    const int fcn = __builtin_amdgcn_readfirstlane(sh_fc[node + 1]);
    const int qr = __builtin_amdgcn_readfirstlane(sh_qrow[max(fcn, 0)]);
    issue_rows(P.target + (trow0 + 1 + node) * static_cast<int64_t>(V),
               fcn >= 0 ? P.draft_q + static_cast<int64_t>(qr) * V : nullptr, sl);
  };
  // The window that begins at a child that is about to be tested: this workgroup's slice of it is fetched while the present
  // round is worked out and its messages travel.  A wrong guess costs its bytes.
  int next_start = -1;                            // first node of the window the rows on their way belong to
  auto chain_node = [&](int start, int steps) {   // the node `steps` first children below, -2 = the chain has ended
    int node = start;
    for (int j = 0; j < steps; ++j) node = node >= -1 ? sh_fc[node + 1] : -2;
    return node;
  };
  auto fetch_ahead = [&](int start) {
    if (U == 0 || start < 0 || start == next_start) return;
    if (next_start >= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // an earlier guess has landed
    next_start = start;
    const int node = chain_node(start, my_lv);
    if (node >= 0) issue_node(node, my_sl);
  };
  auto load_slice = [&](int node, int sl) {
    next_start = -1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (a guess may still be on its way to the same slots)
    issue_node(node, sl);
    settle(sh_fc[node + 1] >= 0, sl);
  };

  auto waves_total = [&](int k) {                 // sum of the waves' sums, the same order everywhere
    double t = sh_ws[k][0];
#pragma unroll
    for (int w = 1; w < kClWaves; ++w) t += sh_ws[k][w];
    return t;
  };

  // Local statistics of the slice in LDS: (max, sum 2^((l - max) c)) of the target part and the draft part.
  // Between two calls (of this or of slice_weight_sum) every wave passes another barrier: what is exchanged here has been read.
  constexpr int N = U ? U : 1;
  float ep[N][8], eq[N][8];                       // U: 2^((l - max of the slice) c), then weights (see weights_to)
  float sl_mp = -INFINITY, sl_mq = -INFINITY;     // ... those maxima
  int held = -1;                                  // ... level of the weights in ep; -1: exponentials
  auto slice_stats = [&](bool have_q, float& mp, double& zp, float& mq, double& zq) {
    float tp = -INFINITY, tq = -INFINITY;
    const int units = data ? UPT : 0;
    if constexpr (U != 0) {
      if (data) {
#pragma unroll
        for (int u = 0; u < N; ++u) { cl_unpack(*row_p(u), ep[u]); cl_unpack(*row_q(u), eq[u]); }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
          for (int j = 0; j < 8; ++j) { tp = fmaxf(tp, ep[u][j]); tq = fmaxf(tq, eq[u][j]); }
      }
    } else {
      for (int u = 0; u < units; ++u) {
        float x[8];
        cl_unpack(*row_p(u), x);
#pragma unroll
        for (int j = 0; j < 8; ++j) tp = fmaxf(tp, x[j]);
        cl_unpack(*row_q(u), x);
#pragma unroll
        for (int j = 0; j < 8; ++j) tq = fmaxf(tq, x[j]);
      }
    }
    cl_max2(tp, tq);
    if (data) { sh_wm[0][wave] = tp; sh_wm[1][wave] = tq; }     // every lane of the wave stores the same value
    cl_sync();
    mp = -INFINITY; mq = -INFINITY;
#pragma unroll
    for (int w = 0; w < kClWaves; w += 4) {
      const float4 a = *reinterpret_cast<const float4*>(&sh_wm[0][w]);
      const float4 b2 = *reinterpret_cast<const float4*>(&sh_wm[1][w]);
      mp = fmaxf(fmaxf(mp, fmaxf(a.x, a.y)), fmaxf(a.z, a.w));
      mq = fmaxf(fmaxf(mq, fmaxf(b2.x, b2.y)), fmaxf(b2.z, b2.w));
    }
    const float sp = (mp == -INFINITY) ? 0.f : mp, sq = (mq == -INFINITY) ? 0.f : mq;
    double ap = 0.0, aq = 0.0;
    if constexpr (U != 0) {
      sl_mp = mp; sl_mq = mq;
      held = -1;
      if (data) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
          float sum = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) { ep[u][j] = fast_exp2((ep[u][j] - sp) * c); sum += ep[u][j]; }
          ap += static_cast<double>(sum);
        }
        if (have_q) {
#pragma unroll
          for (int u = 0; u < N; ++u) {
            float sum = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) { eq[u][j] = fast_exp2((eq[u][j] - sq) * c); sum += eq[u][j]; }
            aq += static_cast<double>(sum);
          }
        }
      }
    } else {
      for (int u = 0; u < units; ++u) {
        float x[8];
        cl_unpack(*row_p(u), x);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += fast_exp2((x[j] - sp) * c);
        ap += static_cast<double>(sum);
        if (have_q) {
          cl_unpack(*row_q(u), x);
          sum = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) sum += fast_exp2((x[j] - sq) * c);
          aq += static_cast<double>(sum);
        }
      }
    }
    cl_sum2(ap, aq);
    if (data) { sh_ws[0][wave] = ap; sh_ws[1][wave] = aq; }
    cl_sync();
    zp = waves_total(0);
    zq = waves_total(1);
  };

  // U: brings ep from the exponentials to the weights of level L (cl_weights says what they are), eq to the draft row's
  // probabilities.  Levels only go up; a level is entered when its mass is known to be positive.
  auto weights_to = [&](const LevelStats& S, int L) {
    if (held < 0) {
      const float m = lane == 0 ? sl_mp : sl_mq, M = lane == 0 ? S.mp : S.mq;
      const double iz = lane == 0 ? S.izp : S.izq;
      // (a row that is -inf throughout is no distribution: its probabilities are NaN, which leaves no residual mass, not 0)
      const float f = m == -INFINITY && M != m ? 0.f : static_cast<float>(cl_exp2(static_cast<double>(m - M) * static_cast<double>(c)) * iz);
      const float fp = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), 0));
      const float fq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), 1));
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) { ep[u][j] *= fp; eq[u][j] *= fq; }
      held = 0;
    }
    for (; held < L; ++held) {
      const float scale = held > 0 ? sh_invRf[held - 1] : 1.f;
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) ep[u][j] = fmaxf(ep[u][j] * scale - eq[u][j], 0.f);
    }
  };

  // Sum of the level-L weights of the held slice (valid in every wave).
  auto slice_weight_sum = [&](const LevelStats& S, int L) -> double {
    double acc = 0.0;
    if constexpr (U != 0) {
      if (data) {
        weights_to(S, L > 0 ? L - 1 : 0);         // (the level itself is not entered: its mass may turn out to be zero)
        const float scale = L > 1 ? sh_invRf[L - 2] : 1.f;
#pragma unroll
        for (int u = 0; u < N; ++u) {
          float sum = 0.f;
#pragma unroll
          for (int j = 0; j < 8; ++j) sum += (L > 0 && held < L) ? fmaxf(ep[u][j] * scale - eq[u][j], 0.f) : ep[u][j];
          acc += static_cast<double>(sum);
        }
      }
    } else {
      for (int u = 0; u < (data ? UPT : 0); ++u) {
        float w[8];
        cl_weights(*row_p(u), *row_q(u), S, c, L, sh_invRf, w);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += w[j];
        acc += static_cast<double>(sum);
      }
    }
    acc = wave_sum(acc);
    if (data) sh_ws[0][wave] = acc;
    cl_sync();
    return waves_total(0);
  };

  // Level-L weights of unit u's classes of this thread.
  auto unit_weights = [&](const LevelStats& S, int L, int u, float (&w)[8]) {
    if constexpr (U != 0) {                       // (slice_parts has brought them to level L)
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (k == u) {
#pragma unroll
          for (int j = 0; j < 8; ++j) w[j] = ep[k][j];
        }
    } else {
      cl_weights(*row_p(u), *row_q(u), S, c, L, sh_invRf, w);
    }
  };

  // Per-(unit, wave) sums of the level-L weights of the held slice, in vocabulary order, for the draw.
  auto slice_parts = [&](const LevelStats& S, int L) {
    cl_sync();
    if (U != 0 && data) weights_to(S, L);
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      if (!data) break;
      float w[8];
      unit_weights(S, L, u, w);
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) sum += w[j];
      const double d = wave_sum(static_cast<double>(sum));
      sh_part[u * kClWaves + wave] = d;
    }
    cl_sync();
  };

  // ---- messages ---- (byte offsets from P.msg, worked out where they are used: kept in registers they end up in scratch
  // memory, and a reload waits behind the message that has just been stored)
  auto msg_at = [&](unsigned r, int wg, int k) { return (((static_cast<unsigned>(b) * 2u + (r & 1u)) * C + wg) * 2u + k) * 32u; };
  auto msg_word = [&](unsigned at) { return reinterpret_cast<unsigned long long*>(reinterpret_cast<unsigned char*>(P.msg) + at); };
  // every lane stores one of the four words (same values from the lanes that share a word)
  auto post = [&](unsigned r, int k, double val, float aux) {
    int l = lane;
    asm volatile("" : "+v"(l));
    const int w = l & 3;
    st_dev(msg_word(msg_at(r, rank, k) + 8u * w), message_word(w, val, aux, P.tag + r));
  };
  // Round r: the wave without logits posts this workgroup's one or two messages and waits for everybody's (the other waves
  // go on to the barrier).  Every wave has passed a barrier since it read what the round before left here.
  // 0: every peer's messages of round r are in sh_val / sh_aux; 1: gave up waiting; 2: the owner walks alone
  auto exchange = [&](unsigned r, int nmsg, double v0, float a0, double v1, float a1) -> int {
    if (!data) {
      post(r, 0, v0, a0);
      if (nmsg == 2) post(r, 1, v1, a1);
      int l = lane;
      asm volatile("" : "+v"(l));
      const int my = min(l, C * nmsg - 1);        // lanes beyond repeat the last message
      const unsigned at = nmsg == 2 ? msg_at(r, my >> 1, my & 1) : msg_at(r, my, 0);
      const int limit = owner ? P.patience : 4 * P.patience + 16;
      int spins = 0, status = -1;
      unsigned long long w[2][kClWords];
      auto look = [&](unsigned long long (&x)[kClWords]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kClWords; ++k) x[k] = ld_dev(msg_word(at + 8u * k));
      };
      auto judge = [&](const unsigned long long (&x)[kClWords]) __attribute__((always_inline)) {     // -1: look again
        const unsigned long long tag = P.tag + r;
        const bool ok = have_tag<kClWords>(x, tag);
        if (__any(have_tag<1>(x, P.tag + kClAbort))) { status = 2; return; }
        if (__all(ok)) {
          status = 0;
          sh_val[my] = message_sum(x);
          sh_aux[my] = message_max<kClWords>(x);
          return;
        }
        if (++spins > 2 * limit) status = 1;      // (two looks take the time of one trip)
      };
      look(w[0]);
      for (;;) {                                  // the next look is on its way while this one is judged
        look(w[1]);
        judge(w[0]);
        if (status >= 0) break;
        look(w[0]);
        judge(w[1]);
        if (status >= 0) break;
      }
      sh_status = status;
    }
    cl_sync();
    return sh_status;
  };

  // ---- the walk; solo: this workgroup computes every slice's part itself ----
  auto walk = [&](const bool solo) -> int {
    int cur = -1, win = -1, depth = 0;            // node the walk is at, first node of the window, tokens accepted
    unsigned r = 0;
    int held_lv = -1, held_sl = -1;               // slice in registers (solo mode)
    auto bring = [&](int lv, int sl) {            // solo: slice sl of level lv of the window, as the workgroup that holds it has it
      const int node = chain_node(win, lv);
      load_slice(node, sl);
      held_lv = lv; held_sl = sl;
      if (U != 0) {
        float mp, mq;
        double zp, zq;
        cl_sync();
        slice_stats(sh_fc[node + 1] >= 0, mp, zp, mq, zq);
        cl_sync();
      }
    };
    for (int guard = 0; guard <= kClNodes + 1; ++guard) {
      // ---- window: the current node and its chain of first children ----
      win = cur;
      ++r;
      if (!solo) {
        const int node = chain_node(win, my_lv);
        float mp = -INFINITY, mq = -INFINITY;
        double zp = 0.0, zq = 0.0;
        // (A later window begins at the child that was fetched ahead last, which waited for the guess before it: what is on its
        // way is this window's, and where this workgroup's level does not exist below that child nothing is.)
        const bool there = guard == 0 ? early : next_start == cur;     // (on its way or here)
        if (node >= -1) {
          if (there) settle(sh_fc[node + 1] >= 0, my_sl);
          else load_slice(node, my_sl);
        }
        next_start = -1;
        if (node >= -1) slice_stats(sh_fc[node + 1] >= 0, mp, zp, mq, zq);
        else cl_sync();
        const int last = chain_node(win, LV - 1);
        fetch_ahead(last >= -1 ? sh_fc[last + 1] : -1);
        const int st = exchange(r, 2, zp, mp, zq, mq);
        if (st) return st;
      } else {
        for (int v = 0; v < C; ++v) {
          const int lv = v / SL, sl = v - lv * SL;
          const int node = chain_node(win, lv);
          float mp = -INFINITY, mq = -INFINITY;
          double zp = 0.0, zq = 0.0;
          if (node >= -1) {
            load_slice(node, sl);
            held_lv = lv; held_sl = sl;
            slice_stats(sh_fc[node + 1] >= 0, mp, zp, mq, zq);
          }
          cl_sync();
          if (wave == 0) { sh_val[2 * v] = zp; sh_aux[2 * v] = mp; sh_val[2 * v + 1] = zq; sh_aux[2 * v + 1] = mq; }
        }
        cl_sync();
      }
      // ---- merge the slices' parts: a wave per (level, row kind), a lane per slice ----
      for (int k = wave; k < 2 * LV; k += kClBlock / kWave) {
        const int lvw = k >> 1, kind = k & 1;
        const bool have = lane < SL;
        const int idx = (lvw * SL + (have ? lane : 0)) * 2 + kind;
        const float m = have ? sh_aux[idx] : -INFINITY;
        const double z = have ? sh_val[idx] : 0.0;
        const float M = wave_max(m);
        const double Z = wave_sum((m == -INFINITY) ? 0.0 : z * cl_exp2(static_cast<double>(m - M) * static_cast<double>(c)));
        sh_M[kind][lvw] = M;                                     // every lane stores the same value
        sh_iZ[kind][lvw] = 1.0 / Z;
      }
      cl_sync();

      // ---- decisions, level by level while the walk follows the chain ----
      int j = 0;
      bool new_window = false;
      while (!new_window) {
        LevelStats S;
        S.mp = sh_M[0][j]; S.izp = sh_iZ[0][j]; S.mq = sh_M[1][j]; S.izq = sh_iZ[1][j];
        int level = 0, sums_level = -1;
        double total = 0.0;

        // one exchange of level-L weight sums of pair j; the slices' sums land in sh_val[j*SL + sl]
        int fail = 0;
        auto sum_round = [&](int L, int candidate) -> double {          // candidate: the child that is tested next, -1 = none
          ++r;
          if (!solo) {
            double mine = 0.0;
            if (my_lv == j) mine = slice_weight_sum(S, L);
            else cl_sync();
            fetch_ahead(candidate);
            const int st = exchange(r, 1, mine, 0.f, 0.0, 0.f);
            if (st) { fail = st; return 0.0; }
          } else {
            for (int sl = 0; sl < SL; ++sl) {
              if (held_lv != j || held_sl != sl) bring(j, sl);
              const double t = slice_weight_sum(S, L);
              cl_sync();
              if (wave == 0) sh_val[j * SL + sl] = t;
            }
            cl_sync();
          }
          // total of the slices' sums (every wave of every workgroup: the same wave-level reduction)
          return wave_sum(lane < SL ? sh_val[j * SL + lane] : 0.0);
        };

        unsigned long long kids = __ballot(my_parent == cur && lane > cur);
        unsigned long long kids_hi = __ballot(my_parent_hi == cur && lane + 64 > cur);
        // p and q of every child's token, each lane its own nodes
        const auto prob = [&](float l, float m, double iz) {
          return cl_exp2((static_cast<double>(l) - static_cast<double>(m)) * static_cast<double>(c)) * iz;
        };
        double lane_p = 0.0, lane_q = 0.0, lane_p_hi = 0.0, lane_q_hi = 0.0;
        if (kids) { lane_p = prob(sh_lp[lane], S.mp, S.izp); lane_q = prob(sh_lq[lane], S.mq, S.izq); }
        if (kids_hi) { lane_p_hi = prob(sh_lp[lane + 64], S.mp, S.izp); lane_q_hi = prob(sh_lq[lane + 64], S.mq, S.izq); }
        int accepted = -1;
        while (kids | kids_hi) {
          int ch;
          if (kids) { ch = __ffsll(static_cast<long long>(kids)) - 1; kids &= kids - 1; }
          else { ch = 64 + __ffsll(static_cast<long long>(kids_hi)) - 1; kids_hi &= kids_hi - 1; }
          const double qx = lane_f64(ch < 64 ? lane_q : lane_q_hi, ch & 63);
          double rx = lane_f64(ch < 64 ? lane_p : lane_p_hi, ch & 63);
          for (int k = 0; k < level; ++k) {
            double w = rx - qx;
            w = w > 0.0 ? w : 0.0;
            rx = w * sh_invR[k];
          }
          if (owner && P.dbg_ratio && wave == 0)
            P.dbg_ratio[o + ch] = static_cast<float>(qx > 0.0 ? rx / qx : (rx > 0.0 ? INFINITY : 0.0));
          // u < r(x) / q(x); q is 0, or NaN where the draft row is no distribution: accepted if r(x) > 0, as on the other paths
          if (qx > 0.0 ? static_cast<double>(sh_u[ch]) * qx < rx : rx > 0.0) { accepted = ch; break; }
          // rejected: mass of max(0, r - q)
          const int sibling = kids ? __ffsll(static_cast<long long>(kids)) - 1 : (kids_hi ? 63 + __ffsll(static_cast<long long>(kids_hi)) : -1);
          const double mass = sum_round(level + 1, sibling);
          if (fail) return fail;
          if (mass > 0.0) {
            const double inv = 1.0 / mass;         // every wave stores the same value and reads its own
            sh_invR[level] = inv; sh_invRf[level] = static_cast<float>(inv);
            ++level;
            sums_level = level;
            total = mass;
          } else {
            sums_level = -1;                       // the residual has no mass: r stays as it was
          }
        }
        if (accepted >= 0) {
          sh_out[depth] = sh_tok[accepted];        // (all waves: the same value)
          ++depth;
          cur = accepted;
          if (j + 1 < LV && chain_node(win, j + 1) == accepted) { ++j; continue; }   // its statistics are in this window
          new_window = true;
          continue;
        }

        // ---- no child, or every child rejected: draw from the level's weights by inverse CDF ----
        if (sums_level != level) {
          total = sum_round(level, -1);
          if (fail) return fail;
        }
        const double target = u_res * total;
        // slice the crossing falls in: inclusive scan of the slices' sums over the lanes (SL <= 32)
        int s_hit;
        double before;
        {
          const double mine = lane < SL ? sh_val[j * SL + lane] : 0.0;
          double inc = mine;
#pragma unroll
          for (int d = 1; d < 32; d <<= 1) {
            const double tq = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += tq;
          }
          unsigned long long hit = __ballot(lane < SL && inc > target);
          if (!hit) hit = __ballot(lane < SL && mine > 0.0) ? (1ull << (63 - __clzll(static_cast<long long>(__ballot(lane < SL && mine > 0.0))))) : 1ull;
          s_hit = __ffsll(static_cast<long long>(hit)) - 1;       // no crossing (rounding): the last slice with positive mass
          before = __shfl(inc - mine, s_hit, kWave);
        }
        if (solo && (held_lv != j || held_sl != s_hit)) bring(j, s_hit);
        if (solo || (my_lv == j && my_sl == s_hit)) {
          slice_parts(S, level);
          // (unit, wave) part the crossing falls in: scan of the parts in vocabulary order (every wave alike)
          int p_hit;
          double run;
          {
            const double a = lane < n_parts ? sh_part[lane] : 0.0;
            double inc_a = a;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
              const double tq = __shfl_up(inc_a, d, kWave);
              if (lane >= d) inc_a += tq;
            }
            const unsigned long long hit_a = __ballot(lane < n_parts && before + inc_a > target);
            const unsigned long long pos_a = __ballot(lane < n_parts && a > 0.0);
            if (hit_a) p_hit = __ffsll(static_cast<long long>(hit_a)) - 1;
            else if (pos_a) p_hit = 63 - __clzll(static_cast<long long>(pos_a));      // rounding: last part with mass
            else p_hit = 0;
            run = before + __shfl(inc_a - a, p_hit, kWave);
          }
          const int u_hit = p_hit / kClWaves, w_hit = p_hit % kClWaves;
          if (wave == w_hit) {
            float w[8];
            unit_weights(S, level, u_hit, w);
            const int e0 = (s_hit * UPT + u_hit) * kClUnit + tid * 8;
            float lsf = 0.f;                       // summed exactly as the parts were
            int my_last = -1;
#pragma unroll
            for (int j2 = 0; j2 < 8; ++j2) { lsf += w[j2]; if (w[j2] > 0.f) my_last = e0 + j2; }
            const double ls = static_cast<double>(lsf);
            double inc = ls;                       // inclusive scan of the lane sums
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
              int tok = -1;
              double acc = run + inc - ls;
#pragma unroll
              for (int j2 = 0; j2 < 8; ++j2) {
                acc += static_cast<double>(w[j2]);
                if (tok < 0 && acc > target && w[j2] > 0.f) tok = e0 + j2;
              }
              if (tok < 0) tok = my_last;          // rounding inside the lane: its last positive class
              found = __shfl(tok, fl, kWave);
            }
            if (found < 0) {                       // rounding across lanes: last positive class of the part
              int ml = my_last;
#pragma unroll
              for (int d = 32; d > 0; d >>= 1) ml = max(ml, __shfl_xor(ml, d, kWave));
              found = ml >= 0 ? ml : min(V - 1, (s_hit * UPT + u_hit) * kClUnit + w_hit * 512);
            }
            if (depth < P.out_stride) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + depth] = found;
          }
        }
        if (owner) {
          if (wave == 0) {
            P.accept_len[b] = depth;
            if (P.stop_node) P.stop_node[b] = cur;
          }
          // (wave 0 alone: it reads what it has stored itself; the token at `depth` is the drawn one)
          for (int i = tid; wave == 0 && i < P.out_stride; i += kWave)
            if (i != depth) P.out_tokens[static_cast<int64_t>(b) * P.out_stride + i] = i < depth ? sh_out[i] : -1;
        }
        return 0;
      }
    }
    return 0;
  };

  bool solo = P.solo != 0;
  for (int attempt = 0; attempt < 2; ++attempt) {
    const int st = walk(solo);
    if (st == 0 || !owner) break;
    // the owner's peers are late or gone: tell them to leave and walk the request alone
    if (wave == 0)
      st_dev(P.msg + ((static_cast<size_t>(b) * 2 + ((lane >> 3) & 1)) * C * 2 + ((lane >> 2) & 1)) * 4 + (lane & 3),
             P.tag + kClAbort);
    cl_sync();
    solo = true;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no slice is on its way to memory that the workgroup gives back
}

ClusterPlan make_cluster_plan(int B, int V, int max_nodes, bool tree, int n_cu, int want_levels, int want_slices) {
  ClusterPlan p{};
  const int units = (V + kClUnit - 1) / kClUnit;
  if (n_cu > 1024) n_cu = 1024;
  int cmax = B > 0 ? n_cu / B : 1;
  cmax = cmax < 1 ? 1 : (cmax > 32 ? 32 : cmax);
  // levels worth speculating on: a linear draft can be accepted to its end; a tree's first-child
  // chain is followed with the probability that first children are accepted
  int lv_need = max_nodes + 1;
  const int lv_cap = tree ? 4 : 9;
  if (lv_need > lv_cap) lv_need = lv_cap;
  // The statistics of a slice are bound by the vector ALU of the one compute unit that holds it, so the
  // slices are made as small as the workgroups available allow; what is left over buys window levels.
  int best_upt = 0, best_lv = 0, best_sl = 0;
  for (int upt = 1; upt <= kClMaxUpt && best_upt == 0; upt *= 2) {
    const int sl = (units + upt - 1) / upt;
    if (upt < 4 && sl > 1 && want_slices <= 0) continue;      // rows are cut into slices of 8192 logits and more
    if (sl > cmax) continue;
    if (want_slices > 0 && sl != want_slices) continue;
    int lv = cmax / sl;
    if (lv > lv_need) lv = lv_need;
    if (want_levels > 0) { if (want_levels * sl > cmax || want_levels > 16) continue; lv = want_levels; }
    best_lv = lv; best_upt = upt; best_sl = sl;
  }
  if (best_upt != 0 && best_lv * best_sl == 1) p.solo = 1;       // a cluster of one exchanges nothing
  if (best_upt == 0) {
    // not even one slice set fits (or the batch exceeds the compute units): one workgroup per request,
    // which computes the parts of ceil(units / 16) slices in turn
    best_upt = kClMaxUpt;
    while (best_upt > 1 && units <= best_upt / 2) best_upt /= 2;
    if (want_slices > 0) {
      for (int upt = 1; upt <= kClMaxUpt; upt *= 2) if ((units + upt - 1) / upt == want_slices) best_upt = upt;
    }
    best_sl = (units + best_upt - 1) / best_upt;
    best_lv = 1;
    p.solo = 1;
  }
  p.upt = best_upt; p.levels = best_lv; p.slices = best_sl;
  return p;
}

size_t cluster_msg_bytes(int B) {
  // (workgroups of all clusters <= B + compute units <= B + 1024) x 2 buffers x 2 messages x 32 bytes
  return (static_cast<size_t>(B) + 1024) * 128;
}

void launch_accept_cluster(const AcceptArgs& a, const ClusterPlan& plan, int patience, void* msg, hipStream_t stream) {
  ClusterParams P;
  P.B = a.B; P.V = a.V; P.n_q_rows = a.n_q_rows > 0 ? a.n_q_rows : 1;
  P.node_offsets = a.node_offsets; P.parent = a.parent; P.draft_tokens = a.draft_tokens;
  P.target = static_cast<const uint16_t*>(a.target);
  P.draft_q = static_cast<const uint16_t*>(a.draft_q);
  P.q_row = a.q_row; P.c = kLog2e / a.temperature; P.u_accept = a.u_accept; P.u_resample = a.u_resample;
  P.accept_len = a.accept_len; P.out_tokens = a.out_tokens; P.out_stride = a.out_stride;
  P.stop_node = a.stop_node; P.dbg_ratio = a.dbg_ratio;
  P.LV = plan.solo ? 1 : plan.levels;
  P.SL = plan.slices;
  P.patience = patience;
  P.solo = plan.solo;
  P.UPT = plan.upt;
  P.msg = static_cast<unsigned long long*>(msg);
  const int C = plan.solo ? 1 : plan.levels * plan.slices;
  // a cluster of one workgroup exchanges nothing: SL stays the number of slices it computes in turn
  const dim3 grid(a.B * C);
  const MessageTag t = plan.solo ? MessageTag{} : next_message_tag(true, stream);
  P.tag = t.tag;
  if (t.clear) clear_messages(P.msg, static_cast<int64_t>(a.B) * C * 16, stream);
  const size_t lds = static_cast<size_t>(plan.upt) * 2 * kClThreads * 16;
  static std::atomic<uint64_t> attr_done{0};
  if (plan.upt == 4) {                            // (32 KB of rows: no attribute needed)
    hipLaunchKernelGGL(accept_cluster_kernel<4>, grid, dim3(kClBlock), lds, stream, P);
    return;
  }
  if (set_lds_once(&accept_cluster_kernel<0>, static_cast<size_t>(kClMaxUpt) * 2 * kClThreads * 16, attr_done) != 0) return;
  hipLaunchKernelGGL(accept_cluster_kernel<0>, grid, dim3(kClBlock), lds, stream, P);
}

}  // namespace specv
