// Attention over the shared paged cache on the matrix cores (bfloat16 cache):
// batches of one- or two-row sequences, and chunks of up to 16 slow rows of
// one sequence (verification, prefill).
//
// What bounds it: the cached keys and values, read once from HBM for all rows
// of a sequence.  The matrix instructions keep the arithmetic out of the way
// (the rows are one operand's 16 columns), and everything between a load and
// its use stays in registers of one wave, so a wave's loop has no barrier and
// a whole next tile is in flight while the current one is multiplied:
//   * a wave takes tiles of 32 tokens.  S^T = K Q^T (rows: tokens): the key
//     rows are read from the cache as the A operand they are (16 bytes per
//     lane), Q^T is the B operand, formed once;
//   * S^T leaves lane (query q = lane % 16, group g = lane / 16) with the
//     scores of tokens 4g..4g+3 of both 16-token halves, which is the B
//     operand of O^T = V^T P^T when the 32 contraction slots are numbered in
//     that order; the softmax's running maximum and sum are then per lane;
//   * lane (n, g) reads 16 bytes (dims 8n..8n+7) of the eight tokens of group
//     g; the 8 x 8 block is transposed in registers (byte permutes) into the
//     A operands of eight products, one for each dim % 8.
// Queries and probabilities are fp32 values cut into three bf16 parts (24
// significant bits, every product exact in fp32), keys and values are bf16 as
// cached: no precision is given up against fp32 arithmetic.
//
// Splits: S_eff = min(S, ceil(ctx / 128)) workgroups of four waves share the
// context of a (sequence, head) by its length now, not by the capacity; the
// last one also forms the rows' own keys and values, writes them to the cache
// and adds their terms; the last to arrive merges the partials.
#pragma once
#include <type_traits>

#include "step_kernels.h"

namespace m2r2 {

constexpr int kMfThreads = 256;
constexpr int kMfWaves = kMfThreads / 64;
constexpr int kMfTile = 32;                        // tokens per wave and tile
constexpr int kMfMinTokens = kMfWaves * kMfTile;   // tokens of a split, at least (while the context has them)
constexpr int kMfMaxTokens = 8192;                 // tokens of a split, at most (its row table is in LDS)

// Tokens a split may hold: ceil(max_ctx / S) in whole tiles.
__host__ __device__ constexpr int mf_split_tokens(int max_ctx, int S) {
  return ((max_ctx + S - 1) / S + kMfTile - 1) / kMfTile * kMfTile;
}
// Dynamic LDS: the row table of a split (S_eff < S only where splits are short).
__host__ __device__ constexpr int mf_attn_lds_bytes(int max_ctx, int S) {
  return 4 * (mf_split_tokens(max_ctx, S) > kMfMinTokens ? mf_split_tokens(max_ctx, S) : kMfMinTokens);
}

// x = h + m + l, each bf16 (round to nearest even): 24 significant bits.
__device__ __forceinline__ void mf_split3(const float (&x)[8], u32x4_t& h, u32x4_t& m, u32x4_t& l) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t hb[2], mb[2], lb[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float v = x[2 * i + k];
      hb[k] = f32_to_bf16_bits(v);
      const float r1 = v - __uint_as_float(hb[k] << 16);
      mb[k] = f32_to_bf16_bits(r1);
      lb[k] = f32_to_bf16_bits(r1 - __uint_as_float(mb[k] << 16));
    }
    h[i] = hb[0] | (hb[1] << 16);
    m[i] = mb[0] | (mb[1] << 16);
    l[i] = lb[0] | (lb[1] << 16);
  }
}

// Infinite or NaN (bf16 bits)?
__device__ __forceinline__ bool mf_odd(uint32_t b) { return (b & 0x7f80u) == 0x7f80u; }

__device__ __forceinline__ f32x4_t mf_mma(u32x4_t a, u32x4_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

// Maximum and sum over the lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float mf_group_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float mf_group_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// One wave's share of a head's attention: up to 16 queries (lane % 16) over
// tiles of 32 tokens.
template <int HD>
struct MfWave {
  static constexpr int NS = HD / 32;   // matrix steps of a score
  static constexpr int ND = HD / 8;    // lanes n that hold dims
  struct Tile {
    u32x4_t k[2][NS], v[8];
  };
  u32x4_t qh[NS], qm[NS], ql[NS];
  float m_run, l_run;   // running maximum of the lane's query, sum over the lane's tokens
  f32x4_t acc[8];       // dim 8 (4 g + i) + j of query q: acc[j][i]

  // q: 8 consecutive floats per step, dims 32 s + 8 g .. (16-byte aligned); zero where not live
  __device__ __forceinline__ void init(const float* q, bool live) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float4 a = *(const float4*)(q + 32 * s + 8 * g), b = *(const float4*)(q + 32 * s + 8 * g + 4);
      float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = live ? x[i] : 0.f;
      mf_split3(x, qh[s], qm[s], ql[s]);
    }
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  static __device__ __forceinline__ u32x4_t ldc(const char* p) {
    return *(const __attribute__((address_space(1))) u32x4_t*)p;
  }
  // tr: cache rows of the tile's 32 tokens; kb, vb: this layer's pages
  static __device__ __forceinline__ void load(const uint32_t* tr, const char* kb, const char* vb, Tile& t) {
    load_k(tr, kb, t);
    load_v(tr, vb, t);
  }
  static __device__ __forceinline__ void load_k(const uint32_t* tr, const char* kb, Tile& t) {
    const int q = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const char* p = kb + (size_t)tr[16 * a + q] * (HD * 2) + 16 * g;
#pragma unroll
      for (int s = 0; s < NS; ++s) t.k[a][s] = ldc(p + 64 * s);
    }
  }
  static __device__ __forceinline__ void load_v(const uint32_t* tr, const char* vb, Tile& t) {
    const int q = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const u32x4_t rows = *(const u32x4_t*)(tr + 16 * a + 4 * g);
#pragma unroll
      for (int x = 0; x < 4; ++x) t.v[4 * a + x] = ldc(vb + (size_t)rows[x] * (HD * 2) + 16 * min(q, ND - 1));
    }
  }

  // see(t): whether the lane's query sees token t of the tile; keys_done()
  // runs once the tile's keys are no longer needed.  FIX: infinite keys are
  // looked for; without, they may leave NaN in l_run
  template <bool FIX, class See>
  __device__ __forceinline__ void tile(const Tile& t, float scale, See see) {
    tile<FIX>(t, scale, see, [] {});
  }
  template <bool FIX, class See, class Done>
  __device__ __forceinline__ void tile(const Tile& t, float scale, See see, Done keys_done) {
    const int g = (threadIdx.x & 63) >> 4;
    f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      s0 = mf_mma(t.k[0][s], ql[s], s0);
      s1 = mf_mma(t.k[1][s], ql[s], s1);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      s0 = mf_mma(t.k[0][s], qm[s], s0);
      s1 = mf_mma(t.k[1][s], qm[s], s1);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      s0 = mf_mma(t.k[0][s], qh[s], s0);
      s1 = mf_mma(t.k[1][s], qh[s], s1);
    }
    // an infinite key times a low part of q that is zero or of the other sign is
    // NaN, the whole product infinite: such a score is its leading parts' alone
    if (FIX && __any(__builtin_isunordered(s0[0], s0[1]) | __builtin_isunordered(s0[2], s0[3]) |
                     __builtin_isunordered(s1[0], s1[1]) | __builtin_isunordered(s1[2], s1[3]))) {
      f32x4_t h0 = {0.f, 0.f, 0.f, 0.f}, h1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        h0 = mf_mma(t.k[0][s], qh[s], h0);
        h1 = mf_mma(t.k[1][s], qh[s], h1);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s0[i] = s0[i] == s0[i] ? s0[i] : h0[i];
        s1[i] = s1[i] == s1[i] ? s1[i] : h1[i];
      }
    }
    keys_done();
    float z[8], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int tok = (i < 4 ? 0 : 16) + 4 * g + (i & 3);
      z[i] = see(tok) ? (i < 4 ? s0[i & 3] : s1[i & 3]) * scale : -INFINITY;
      mx = fmaxf(mx, z[i]);
    }
    const float mn = fmaxf(m_run, mf_group_max(mx));
    const float al = m_run == -INFINITY ? 0.f : __expf(m_run - mn);
    m_run = mn;
    float p[8], ls = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      p[i] = z[i] == -INFINITY ? 0.f : __expf(z[i] - mn);
      ls += p[i];
    }
    l_run = l_run * al + ls;
    if (__any(al != 1.f)) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] *= al;
    }
    u32x4_t ph, pm, pl;
    mf_split3(p, ph, pm, pl);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // dim 8 n + j of the lane's eight tokens
      u32x4_t vt;
#pragma unroll
      for (int w = 0; w < 4; ++w)
        vt[w] = __builtin_amdgcn_perm(t.v[2 * w + 1][j >> 1], t.v[2 * w][j >> 1], (j & 1) ? 0x07060302u : 0x05040100u);
      acc[j] = mf_mma(vt, pl, acc[j]);
      acc[j] = mf_mma(vt, pm, acc[j]);
      acc[j] = mf_mma(vt, ph, acc[j]);
    }
  }

  // Query q's maximum and sum, and its accumulators (HD floats at `out`, 16-byte aligned).
  __device__ __forceinline__ void store(bool live, float* m, float* l, float* out) {
    const int g = (threadIdx.x & 63) >> 4;
    const float ls = mf_group_sum(l_run);
    if (!live) return;
    if (g == 0) {
      *m = m_run;
      *l = ls;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = 4 * g + i;
      if (n < ND) {
        *(float4*)(out + 8 * n) = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
        *(float4*)(out + 8 * n + 4) = make_float4(acc[4][i], acc[5][i], acc[6][i], acc[7][i]);
      }
    }
  }
};

// RMAX: rows of a sequence, at most: 2 (slow and fast row, or one row alone) or 16 (a chunk of slow rows).
template <int WB, int HD, int RMAX>
__global__ __launch_bounds__(kMfThreads, 2) void km_attn(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io, KVPtrs kv,
                                                         int layer, int S) {
  constexpr int NS = HD / 32;     // matrix steps of a score
  constexpr int ND = HD / 8;      // lanes that hold dims (n < ND)
  constexpr int HALF = HD / 2;
  constexpr int QP = HD + 4;      // padded row of q (floats)
  constexpr int NQ = (RMAX * HALF + kMfThreads - 1) / kMfThreads;        // pairs (j, j + HD/2) of q per thread
  constexpr int NKV = (2 * RMAX * HALF + kMfThreads - 1) / kMfThreads;   // and of k and v
  constexpr bool DUAL = RMAX == 2;                                       // the last row may be a fast row
  static_assert(HD % 32 == 0 && ND <= 16, "head dim");
  extern __shared__ __attribute__((aligned(16))) uint32_t trow[];   // cache row of every token of the split
  __shared__ __attribute__((aligned(16))) float q_s[16][QP];
  __shared__ __attribute__((aligned(16))) uint16_t ko_s[16][HD], vo_s[16][HD];   // own keys, values as cached
  __shared__ float kf_s[HD], vf_s[HD];               // the fast row's own key and value, exact
  __shared__ __attribute__((aligned(16))) float acc_s[kMfWaves][RMAX][HD];
  __shared__ float m_s[kMfWaves][16], l_s[kMfWaves][16];
  __shared__ float mw[RMAX][64], lw[RMAX][64], linv[RMAX];
  __shared__ float u_s[3 * kMaxRank];
  __shared__ float ownf_s;
  __shared__ float uop[DUAL ? kMaxRank * (HD / 8) : 1];
  __shared__ u32x4_t ao_s[DUAL ? kMaxRank * (HD / 8) : 1];   // A_o of the head, 8 columns each (bf16 weights)
  __shared__ int bt_s[kMfThreads];                           // first entries of the block table
  __shared__ SkRmLds rmu;
  __shared__ int last_flag, odd_s;   // odd_s: a slow row's own value is infinite or NaN
  const RowMap& rml = rmu.rm;
  const int h = blockIdx.x, sq = blockIdx.y, sp = blockIdx.z;   // working splits are dispatched first
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int q = lane & 15, g = lane >> 4;
  const int r = D.r, qd = D.qdim, nqkv = 3 * qd + 3 * r;

  // first row and row count of the sequence, and whether its last row is a
  // fast one (scalars: constant-index reads of the map, uniform selects)
  int first = rm.first[0], R = rm.cnt[0];
#pragma unroll
  for (int i = 1; i < kMaxSeq; ++i) {
    first = sq == i ? (int)rm.first[i] : first;
    R = sq == i ? (int)rm.cnt[i] : R;
  }
  const int fast_i = DUAL && rsel(rm.fast, first + R - 1) ? R - 1 : -1;

  // ---- round one: everything that does not depend on the position ----------
  const int posv = io.positions[sq];
  const int exv = ws.exited[sq];
  const int btv = kv.bt[sq * kv.mbps + min(tid, kv.mbps - 1)];
  const int nq = R * HALF;
  float qa[NQ], qb[NQ];
#pragma unroll
  for (int it = 0; it < NQ; ++it) {
    const int e = min(tid + it * kMfThreads, nq - 1);
    const float* src = ws.QKV + (size_t)(first + e / HALF) * nqkv + h * HD + e % HALF;
    qa[it] = src[0];
    qb[it] = src[HALF];
  }
  // the fast row: adapter-down sums, its rows of B_q (k, v: threads of the own
  // split only, later), A_o of the head
  float uv = 0.f;
  u32x4_t bq[2][2];
  constexpr int NAO = (kMaxRank * ND + kMfThreads - 1) / kMfThreads;
  u32x4_t ao[NAO];
  const bool b16 = WB && DUAL && (r == 8 || r == 16);   // B rows of one or two 16-byte pieces
  if constexpr (DUAL) {
    const int fm = first + max(fast_i, 0);
    uv = ws.QKV[(size_t)fm * nqkv + 3 * qd + min(tid, 3 * r - 1)];
    if (b16 && fast_i >= 0 && L.A[0] && L.B[0]) {
      const int j = tid % HALF;
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int k = 0; k < 2; ++k)
          bq[x][k] = ((const u32x4_t*)L.B[0])[((size_t)h * HD + j + x * HALF) * (r / 8) + min(k, r / 8 - 1)];
    }
    if (WB && fast_i >= 0 && L.A[3]) {
#pragma unroll
      for (int k = 0; k < NAO; ++k) {
        const int e = min(tid + k * kMfThreads, r * ND - 1);
        ao[k] = *(const u32x4_t*)((const uint16_t*)L.A[3] + (size_t)(e / ND) * qd + h * HD + 8 * (e % ND));
      }
    }
  }
  // ---- the position (requested first) decides which tokens are this split's;
  // a split beyond the context leaves without waiting for the rest ----------------
  __builtin_amdgcn_sched_barrier(0);
  const int pos0 = posv + rm.pos_offset;
  const bool frozen = exv != 0;
  const int ctx = max(0, min(pos0, min(ws.rope_len, kv.mbps * kv.bs)));
  const int s_eff = max(1, min(S, (ctx + kMfMinTokens - 1) / kMfMinTokens));
  const bool own = sp == s_eff - 1;
  if (sp >= s_eff || (frozen && !own)) return;   // an exited sequence only writes its cache entries
  __builtin_amdgcn_sched_barrier(0);
  sk_rm_copy(rmu, rm);
  bt_s[tid] = btv;
  if (tid == 0) odd_s = 0;
  if constexpr (DUAL) {
    if (tid < 3 * r) u_s[tid] = uv;
    if (WB && fast_i >= 0 && L.A[3]) {
#pragma unroll
      for (int k = 0; k < NAO; ++k)
        if (tid + k * kMfThreads < r * ND) ao_s[tid + k * kMfThreads] = ao[k];
    }
  }
  // zero what the operands read beyond the rows
  for (int e = tid; e < 16 * QP; e += kMfThreads)
    if (e / QP >= R) q_s[e / QP][e % QP] = 0.f;
  __syncthreads();

  const int per = mf_split_tokens(ctx, s_eff);
  const int t0 = min(ctx, sp * per), nt = min(ctx, t0 + per) - t0;
  const int ntile = (nt + kMfTile - 1) / kMfTile;
  auto row_of = [&](int tp) -> int64_t {   // the row's cache row of this layer and head, -1 outside the table
    const int lb = tp / kv.bs;
    if (tp < 0 || lb >= kv.mbps) return -1;
    const int b = lb < kMfThreads ? bt_s[lb] : kv.bt[sq * kv.mbps + lb];
    if (b < 0 || b >= kv.num_blocks) return -1;
    return ((int64_t)b * D.H + h) * kv.bs + (tp - lb * kv.bs);
  };
  // cache rows of the split's tokens; the last tile is filled up with the last
  // token's row (masked in the scores)
  for (int j = tid; j < ntile * kMfTile; j += kMfThreads) {
    const int64_t row = row_of(t0 + min(j, nt - 1));
    trow[j] = row < 0 ? (uint32_t)(h * kv.bs) : (uint32_t)row;
  }
  // RoPE entries; in the own split the projections to k and v
  auto rope_at = [&](int i, int j) {
    int pos = pos0 + rml.idx[first + i];
    if (pos < 0 || pos >= ws.rope_len) {
      atomicOr(ws.err, 8);
      pos = 0;
    }
    return ws.rope[(size_t)pos * HALF + j];
  };
  float2 cq[NQ];
#pragma unroll
  for (int it = 0; it < NQ; ++it) {
    const int e = min(tid + it * kMfThreads, nq - 1);
    cq[it] = rope_at(e / HALF, e % HALF);
  }
  float va0[NKV], vb0[NKV];
  float2 ck[NKV];
  u32x4_t bkv[2][2];   // the fast row's rows of B_k or B_v (NKV is 1)
  const int nkv = own ? 2 * nq : 0;
#pragma unroll
  for (int it = 0; it < NKV; ++it) {
    if (it * kMfThreads >= nkv) break;   // (uniform)
    const int e = min(tid + it * kMfThreads, nkv - 1);
    const int w = 1 + e / nq, i = (e % nq) / HALF, j = e % HALF;
    const float* src = ws.QKV + (size_t)(first + i) * nqkv + w * qd + h * HD + j;
    va0[it] = src[0];
    vb0[it] = src[HALF];
    ck[it] = rope_at(i, j);
    if constexpr (DUAL) {
      const void* B = w == 1 ? L.B[1] : L.B[2];
      if (b16 && i == fast_i && B) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int k = 0; k < 2; ++k)
            bkv[x][k] = ((const u32x4_t*)B)[((size_t)h * HD + j + x * HALF) * (r / 8) + min(k, r / 8 - 1)];
      }
    }
  }
  if (own)
    for (int e = tid; e < 16 * HD; e += kMfThreads)
      if (e / HD >= R) ko_s[e / HD][e % HD] = vo_s[e / HD][e % HD] = 0;
  __syncthreads();
  // ---- the first tile's keys and values, in flight while q is formed ---------
  const size_t lay0 = (size_t)layer * kv.num_blocks * D.H * kv.bs;
  const char* kb = (const char*)kv.k + lay0 * HD * 2;
  const char* vb = (const char*)kv.v + lay0 * HD * 2;
  using MW = MfWave<HD>;
  typename MW::Tile ta, tb;
  int tt = wv;
  if (!frozen && tt < ntile) MW::load(trow + tt * kMfTile, kb, vb, ta);
  __builtin_amdgcn_sched_barrier(0);
  // adapter-up of a fast row's pair of projection w (pre: its rows of B, loaded)
  auto adapt = [&](int w, int j, const u32x4_t (&pre)[2][2], float& a, float& b) {
    const void* B = w == 0 ? L.B[0] : (w == 1 ? L.B[1] : L.B[2]);
    const void* A = w == 0 ? L.A[0] : (w == 1 ? L.A[1] : L.A[2]);
    if (!A || !B) return;
    const float* u = u_s + w * r;
    if (b16) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (8 * k >= r) break;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float u0 = u[8 * k + 2 * x], u1 = u[8 * k + 2 * x + 1];
          a += bf16lo(pre[0][k][x]) * u0 + bf16hi(pre[0][k][x]) * u1;
          b += bf16lo(pre[1][k][x]) * u0 + bf16hi(pre[1][k][x]) * u1;
        }
      }
    } else {
      a += dot_row_t<WB>(B, (size_t)h * HD + j, r, u);
      b += dot_row_t<WB>(B, (size_t)h * HD + j + HALF, r, u);
    }
  };
#pragma unroll
  for (int it = 0; it < NQ; ++it) {
    const int e = tid + it * kMfThreads;
    if (e >= nq) break;
    const int i = e / HALF, j = e % HALF;
    float a = qa[it], b = qb[it];
    if (DUAL && i == fast_i) adapt(0, j, bq, a, b);
    q_s[i][j] = a * cq[it].x - b * cq[it].y;
    q_s[i][j + HALF] = b * cq[it].x + a * cq[it].y;
  }
#pragma unroll
  for (int it = 0; it < NKV; ++it) {
    const int e = tid + it * kMfThreads;
    if (e >= nkv) break;
    const int w = 1 + e / nq, i = (e % nq) / HALF, j = e % HALF;
    float a = va0[it], b = vb0[it];
    if (DUAL && i == fast_i) adapt(w, j, bkv, a, b);
    if (w == 1) {
      const float x = a * ck[it].x - b * ck[it].y, y = b * ck[it].x + a * ck[it].y;
      a = x;
      b = y;
    }
    uint16_t* o = w == 1 ? &ko_s[i][0] : &vo_s[i][0];
    o[j] = (uint16_t)f32_to_bf16_bits(a);
    o[j + HALF] = (uint16_t)f32_to_bf16_bits(b);
    if (w == 2 && i != fast_i && (mf_odd(o[j]) || mf_odd(o[j + HALF]))) odd_s = 1;
    if (DUAL && i == fast_i) {
      float* f = w == 1 ? kf_s : vf_s;
      f[j] = a;
      f[j + HALF] = b;
    }
  }
  __syncthreads();
  // ---- own split: cache writes, 16 bytes per thread --------------------------
  if (own) {
    for (int e = tid; e < 2 * R * ND; e += kMfThreads) {
      const int w = e / (R * ND), i = (e / ND) % R, c = e % ND;
      if (!rml.wr[first + i]) continue;
      const int64_t row = row_of(pos0 + rml.idx[first + i]);
      if (row < 0) {
        atomicOr(ws.err, 2);
        continue;
      }
      const size_t ix = (lay0 + (size_t)row) * HD + 8 * c;
      *(u32x4_t*)((uint16_t*)(w ? kv.v : kv.k) + ix) = *(const u32x4_t*)(w ? &vo_s[i][8 * c] : &ko_s[i][8 * c]);
    }
  }
  if (frozen) return;
  const float scale = rsqrtf((float)HD);
  if (DUAL && own && fast_i >= 0 && wv == kMfWaves - 1) {   // the fast row's own score, exact key
    float p = 0.f;
    for (int d = lane; d < HD; d += 64) p += q_s[fast_i][d] * kf_s[d];
    p = wave_sum(p);
    if (lane == 0) ownf_s = p * scale;
  }
  MW mw_;
  mw_.init(q_s[q], true);   // (rows beyond the sequence's are zero)
  while (tt < ntile) {
    if (tt + kMfWaves < ntile) MW::load(trow + (tt + kMfWaves) * kMfTile, kb, vb, tb);
    mw_.template tile<false>(ta, scale, [left = nt - tt * kMfTile](int t) { return t < left; });
    tt += kMfWaves;
    if (tt >= ntile) break;
    if (tt + kMfWaves < ntile) MW::load(trow + (tt + kMfWaves) * kMfTile, kb, vb, ta);
    mw_.template tile<false>(tb, scale, [left = nt - tt * kMfTile](int t) { return t < left; });
    tt += kMfWaves;
  }
  const bool own_wave = own && wv == (ntile & (kMfWaves - 1));
  auto own_tile = [&](auto fix) {
    // the rows' own keys: a slow row sees the slow rows up to itself, as cached
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      ta.k[0][s] = *(const u32x4_t*)&ko_s[q][32 * s + 8 * g];
      ta.k[1][s] = u32x4_t{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      // (the products take every row's values, those not seen times zero:
      // infinities and NaN stay out and are added below where they are seen)
      ta.v[t] = *(const u32x4_t*)&vo_s[4 * g + t][8 * min(q, ND - 1)];
      if (4 * g + t == fast_i) ta.v[t] = u32x4_t{0u, 0u, 0u, 0u};
      if (odd_s) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
          ta.v[t][x] &= (mf_odd(ta.v[t][x]) ? 0u : 0xffffu) | (mf_odd(ta.v[t][x] >> 16) ? 0u : 0xffff0000u);
      }
      ta.v[4 + t] = u32x4_t{0u, 0u, 0u, 0u};
    }
    const bool slow = q < R && q != fast_i;
    mw_.template tile<decltype(fix)::value>(ta, scale, [&](int t) { return slow && t <= q && t != fast_i; });
  };
  if (own_wave) own_tile(std::false_type{});
  // A NaN score (an infinite key, perhaps): once more, with such keys looked
  // for (in the loop above that costs eight sequences of 4096 positions 1.6 us a layer)
  if (__any(mw_.l_run != mw_.l_run)) {
    mw_.init(q_s[q], true);
    for (tt = wv; tt < ntile; tt += kMfWaves) {
      MW::load(trow + tt * kMfTile, kb, vb, ta);
      mw_.template tile<true>(ta, scale, [left = nt - tt * kMfTile](int t) { return t < left; });
    }
    if (own_wave) own_tile(std::true_type{});
  }
  // ---- the waves' results, combined --------------------------------------------
  mw_.store(q < R, &m_s[wv][q], &l_s[wv][q], acc_s[wv][min(q, RMAX - 1)]);
  __syncthreads();
  const int stride = 2 + HD + r;
  float* part = ws.att + (((size_t)sq * D.H + h) * (S + 1)) * kMaxRows * stride;
  for (int e = tid; e < R * HD; e += kMfThreads) {
    const int i = e / HD, d = e % HD;
    const bool of = DUAL && own && i == fast_i;
    float M = of ? ownf_s : -INFINITY;
#pragma unroll
    for (int w = 0; w < kMfWaves; ++w) M = fmaxf(M, m_s[w][i]);
    const float wo = of ? __expf(ownf_s - M) : 0.f;
    float a = of ? wo * vf_s[d] : 0.f, l = wo;
#pragma unroll
    for (int w = 0; w < kMfWaves; ++w) {
      const float x = l_s[w][i] > 0.f ? __expf(m_s[w][i] - M) : 0.f;
      a += x * acc_s[w][i][d];
      l += x * l_s[w][i];
    }
    if (own && odd_s && i != fast_i) {
      for (int t = 0; t <= i; ++t)
        if (t != fast_i && mf_odd(vo_s[t][d])) a += __uint_as_float((uint32_t)vo_s[t][d] << 16);
    }
    if (s_eff == 1) {
      const float o = a / l;
      put_o(D, rm, ws, first + i, h * HD + d, o);
      q_s[i][d] = o;
    } else {
      float* pp = part + ((size_t)sp * kMaxRows + i) * stride;
      st_agent(pp + 2 + d, a);
      if (d == 0) {
        st_agent(pp, M);
        st_agent(pp + 1, l);
      }
    }
  }
  // ---- the last split to arrive merges -----------------------------------------
  if (s_eff > 1) {
    if (!arrive_last(&ws.att_cnt[sq * D.H + h], s_eff, &last_flag)) return;
    for (int e = tid; e < R * s_eff; e += kMfThreads) {
      const int i = e / s_eff, s2 = e % s_eff;
      const float* pp = part + ((size_t)s2 * kMaxRows + i) * stride;
      mw[i][s2] = ld_agent(pp);
      lw[i][s2] = ld_agent(pp + 1);
    }
    constexpr int NE = (RMAX * HD + kMfThreads - 1) / kMfThreads;
    // the first splits' accumulators are requested with the weights
    constexpr int PF = DUAL ? 8 : 4;
    float pv[NE][PF];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int e = min(tid + k * kMfThreads, R * HD - 1);
#pragma unroll
      for (int u = 0; u < PF; ++u)
        pv[k][u] = ld_agent(part + ((size_t)min(u, s_eff - 1) * kMaxRows + e / HD) * stride + 2 + e % HD);
    }
    __syncthreads();
    if (tid < R) {
      float M = -INFINITY, Ls = 0.f;
      for (int s2 = 0; s2 < s_eff; ++s2)
        if (lw[tid][s2] > 0.f) M = fmaxf(M, mw[tid][s2]);
      for (int s2 = 0; s2 < s_eff; ++s2) {
        const float w = lw[tid][s2] > 0.f ? __expf(mw[tid][s2] - M) : 0.f;
        mw[tid][s2] = w;
        Ls += w * lw[tid][s2];
      }
      linv[tid] = 1.f / Ls;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int e = tid + k * kMfThreads;
      if (e >= R * HD) break;
      const int i = e / HD, d = e % HD;
      float v = 0.f;
#pragma unroll
      for (int u = 0; u < PF; ++u)
        if (u < s_eff) v += mw[i][u] * pv[k][u];
#pragma unroll 4
      for (int u = PF; u < s_eff; ++u) v += mw[i][u] * ld_agent(part + ((size_t)u * kMaxRows + i) * stride + 2 + d);
      v *= linv[i];
      put_o(D, rm, ws, first + i, h * HD + d, v);
      q_s[i][d] = v;
    }
  }
  if constexpr (DUAL) {
    // o-adapter share of this head: uo[row][h][j] = sum_d A_o[j][h HD + d] o[d] (fast rows; 0 else)
    __syncthreads();
    const bool ad = fast_i >= 0 && L.A[3];
    if (ad) {
      for (int e = tid; e < r * ND; e += kMfThreads) {
        const float* o = &q_s[fast_i][8 * (e % ND)];
        float a = 0.f;
        if constexpr (WB) {
#pragma unroll
          for (int x = 0; x < 4; ++x) a += bf16lo(ao_s[e][x]) * o[2 * x] + bf16hi(ao_s[e][x]) * o[2 * x + 1];
        } else {
          const size_t base = (size_t)(e / ND) * qd + h * HD + 8 * (e % ND);
#pragma unroll
          for (int x = 0; x < 8; ++x) a += ld_wt<WB>(L.A[3], base + x) * o[x];
        }
        uop[e] = a;
      }
      __syncthreads();
    }
    for (int e = tid; e < R * r; e += kMfThreads) {
      const int i = e / r, j = e % r;
      float a = 0.f;
      if (ad && i == fast_i)
        for (int c = 0; c < ND; ++c) a += uop[j * ND + c];
      ws.uo[((size_t)(first + i) * D.H + h) * r + j] = a;
    }
  }
}

}  // namespace m2r2
