// Projections of passes with 3 to 16 rows, bfloat16 weights (batched decoding,
// verification chunks, prefill): kt_qkv, kt_oproj, kt_gateup, kt_down, kt_head.
//
// What bounds them: the weights, read once from HBM for all rows; at 16 rows
// the matrix instructions need a tenth of that time.  So the design keeps
// every compute unit's loads in flight from its first cycle to its last and
// does as little as possible between them:
//   * One workgroup of 8 waves per compute unit (up to 256 registers per
//     lane).  A tile is `th` weight rows; the waves split its reduction.  th
//     is 16, or 12 where that spreads the rows evenly over the compute units
//     (d = 3072 over 256: 12 each instead of 16 on three quarters of them).
//   * The activations are read as the matrix operands they are: the producing
//     kernel leaves them as bf16 hi + lo parts (16 significant bits of the
//     fp32 value, the norm gain already applied) in operand order, 2 KB per 32
//     elements of reduction ("planes").  Up to 3072 elements a wave holds its
//     share in registers for all its tiles; longer reductions stream it
//     beside the weights.  (Reading fp32 rows and cutting them per tile moved
//     twice the bytes of the weights through the L1.)
//   * Up to 8 rows, the hi and lo parts are the two halves of one operand's
//     16 rows: one matrix instruction per step instead of two.
//   * The next tile's weights are requested before the current one is
//     multiplied, and the partial sums of up to four tiles are added through
//     LDS in one step, so the workgroup meets at two barriers per four tiles.
#pragma once
#include "step_kernels.h"

namespace m2r2 {

constexpr int kTpWaves = 8;
constexpr int kTpThreads = kTpWaves * 64;
constexpr int kTpTiles = 4;     // tiles whose sums are added together
constexpr int kTpRedCol = 20;   // floats per column of a wave's partial tile (16 rows, padded)

// Bytes of the planes of 16 rows of K elements.
__host__ __device__ constexpr size_t tp_plane_bytes(int K) { return (size_t)(K + 31) / 32 * 2048; }

// Tile-packed weights with th rows per tile: the block of step s of a tile is
// th * 64 bytes, [4][th][8] elements (k group, row, element).
__global__ __launch_bounds__(256) void k_pack_th(PackSrc src, int total_rows, int K, int th, void* dst) {
  const int S = K / 32;
  const size_t per = (size_t)S * 4 * th;   // 16-byte pieces per tile
  const size_t n = (size_t)((total_rows + th - 1) / th) * per;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t t = i / per;
    const int rem = (int)(i - t * per), s = rem / (4 * th), gr = rem % (4 * th);
    int r = (int)t * th + gr % th;
    const int col = s * 32 + 8 * (gr / th);
    u32x4_t v = {0u, 0u, 0u, 0u};
    for (int g = 0; g < 3; ++g) {
      if (r < src.rows[g]) {
        if (src.p[g]) v = *(const u32x4_t*)((const char*)src.p[g] + ((size_t)r * K + col) * 2);
        break;
      }
      r -= src.rows[g];
    }
    *(u32x4_t*)((char*)dst + i * 16) = v;
  }
}

// 16-byte load: scalar base, this lane's offset, scalar offset.
__device__ __forceinline__ u32x4_t tp_ld(const char* base, int lane_off, size_t off) {
  return *(const __attribute__((address_space(1))) u32x4_t*)(base + off + lane_off);
}
__device__ __forceinline__ u32x4_t tp_ld_w(const char* base, int lane_off, size_t off) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_t*)(base + off + lane_off));
}

// NS > 0: a wave's share of the reduction is at most NS steps of 32, its
// activations stay in registers.  NS == 0: any length, streamed.  T: tiles
// whose sums are added together (1: usually the workgroup's only tile, so a
// next one is not requested ahead).
template <int NS, int MT, int T>
struct TpCore {
  static constexpr int NP = MT > 8 ? 2 : 1;      // activation operands per step
  static constexpr bool RES = NS > 0;
  static constexpr int CS = 4, PD = 4;           // streamed: steps per chunk, chunks in flight
  static constexpr int NW = RES ? (T > 1 ? 2 : 1) : PD;        // weight buffers
  static constexpr int SW = RES ? NS : CS;       // steps of a buffer
  static constexpr int NA = RES ? 1 : PD;        // activation buffers
  u32x4_t w[NW][SW];
  u32x4_t a[NA][SW][NP];
  const char* x;       // planes
  int s0, s1;          // this wave's steps
  int xo, wo;          // lane offsets
  int blk;
  int nch;             // streamed: chunks of a tile, a multiple of PD

  // block: bytes from a step's block of a tile to the next step's
  // split: this workgroup's part of the reduction, of n_split equal ones
  __device__ __forceinline__ void init(int K, int tile_rows, int block, const uint16_t* planes, int split = 0,
                                       int n_split = 1) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, g = lane >> 4;
    const int nsteps = K / 32 / n_split, per = (nsteps + kTpWaves - 1) / kTpWaves;
    const int b0 = split * nsteps;
    s0 = b0 + min(nsteps, wave * per);
    s1 = min(b0 + nsteps, s0 + per);
    x = (const char*)planes;
    const int th = tile_rows;
    blk = block;
    wo = (g * th + min(row, th - 1)) * 16;
    xo = MT > 8 ? (g * 16 + row) * 16 : ((row >> 3) * 64 + g * 16 + (row & 7)) * 16;
    nch = (per + CS * PD - 1) / (CS * PD) * PD;
  }
  // steps past the range repeat its last one (a cache hit; their activations are zeroed)
  __device__ __forceinline__ int step_of(int s) const { return max(min(s, s1 - 1), 0); }

  __device__ __forceinline__ void load_a(int sb, u32x4_t (&dst)[SW][NP], bool live = true) const {
#pragma unroll
    for (int j = 0; j < SW; ++j)
#pragma unroll
      for (int p = 0; p < NP; ++p)
        dst[j][p] = tp_ld(x, xo, (size_t)(live ? step_of(sb + j) : step_of(s0)) * 2048 + p * 1024);
  }
  __device__ __forceinline__ void load_w(const char* tile, int sb, bool live, u32x4_t (&dst)[SW]) const {
    // (not live: nothing left to stream; the loads stay, of one block)
#pragma unroll
    for (int j = 0; j < SW; ++j) dst[j] = tp_ld_w(tile, wo, (size_t)(live ? step_of(sb + j) : step_of(s0)) * blk);
  }
  __device__ __forceinline__ void zero_tail(int sb, u32x4_t (&v)[SW][NP]) const {
#pragma unroll
    for (int j = 0; j < SW; ++j)
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (sb + j >= s1) v[j][p] = u32x4_t{0u, 0u, 0u, 0u};
  }

  // Request the activations and the first weights.
  template <class Ptr>
  __device__ __forceinline__ void begin(int n_local, const Ptr& ptr) {
    if constexpr (RES) {
      load_a(s0, a[0]);
      __builtin_amdgcn_sched_barrier(0);
      load_w(ptr(0), s0, true, w[0]);
      if constexpr (T > 1) load_w(ptr(min(1, n_local - 1)), s0, n_local > 1, w[1]);
    } else {
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        load_a(s0 + u * CS, a[u]);
        load_w(ptr(0), s0 + u * CS, true, w[u]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // The same where the rows are not known yet: the first weights, then (once
  // they are) the activations and, behind them, the next tile's weights.
  template <class Ptr>
  __device__ __forceinline__ void begin_w(const Ptr& ptr) {
#pragma unroll
    for (int u = 0; u < (RES ? 1 : PD); ++u) load_w(ptr(0), s0 + u * CS, true, w[u]);
    __builtin_amdgcn_sched_barrier(0);
  }
  // take: this lane reads the row before its own
  template <class Ptr>
  __device__ __forceinline__ void begin_x(int n_local, const Ptr& ptr, bool take) {
    if (take) xo -= 16;
#pragma unroll
    for (int u = 0; u < NA; ++u) load_a(s0 + u * CS, a[u]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (RES && T > 1) load_w(ptr(min(1, n_local - 1)), s0, n_local > 1, w[1]);
    __builtin_amdgcn_sched_barrier(0);
  }

  __device__ __forceinline__ void mul(const u32x4_t (&av)[SW][NP], const u32x4_t (&wv)[SW], f32x4_t& acc) const {
#pragma unroll
    for (int j = 0; j < SW; ++j)
#pragma unroll
      for (int p = 0; p < NP; ++p)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av[j][p]),
                                                      __builtin_bit_cast(bf16x8_t, wv[j]), acc, 0, 0, 0);
  }

  // Stream the workgroup's tiles; after every T of them (and the last)
  // epi(base, count) finds their per-wave sums in `red`.  Refills are made
  // unconditionally (a load under a branch would make the waits behind it wait
  // for everything in flight); with nothing left they repeat one block.
  template <class Ptr, class Epi>
  __device__ __forceinline__ void run(int n_local, const Ptr& ptr, float* red, Epi&& epi) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if constexpr (RES) zero_tail(s0, a[0]);
    for (int base = 0; base < n_local; base += T) {
      f32x4_t acc[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (T > 1 && base + t >= n_local) continue;   // (uniform)
        if constexpr (RES) {
          static_assert(T == 1 || T % 2 == 0, "buffers alternate");
          mul(a[0], w[t % NW], acc[t]);
          if constexpr (T == 1) {
            if (base + 1 < n_local) load_w(ptr(base + 1), s0, true, w[0]);   // (uniform)
          } else {
            const bool more = base + t + 2 < n_local;
            load_w(ptr(more ? base + t + 2 : base + t), s0, more, w[t % NW]);
          }
        } else {
          for (int c = 0; c < nch; c += PD) {
            const bool next = c + PD >= nch;   // refills belong to the next tile
            const bool more = !next || base + t + 1 < n_local;
            const char* np = ptr(next && more ? base + t + 1 : base + t);
#pragma unroll
            for (int u = 0; u < PD; ++u) {
              zero_tail(s0 + (c + u) * CS, a[u]);
              mul(a[u], w[u], acc[t]);
              const int sb = s0 + (next ? u : c + PD + u) * CS;
              load_a(sb, a[u], more);
              load_w(np, sb, more, w[u]);
            }
          }
        }
      }
      if (base > 0) __syncthreads();   // the sums of the group before have been read
#pragma unroll
      for (int t = 0; t < T; ++t)
        *(f32x4_t*)(red + ((wave * T + t) * 16 + (lane & 15)) * kTpRedCol + 4 * (lane >> 4)) = acc[t];
      __syncthreads();
      epi(base, min(T, n_local - base));
    }
  }
};

// Sum of row m, column n of tile t over the waves (and hi and lo rows).
template <int MT, int T>
__device__ __forceinline__ float tp_sum(const float* red, int t, int m, int n) {
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kTpWaves; ++w) {
    const float* p = red + ((w * T + t) * 16 + n) * kTpRedCol + m;
    s += MT > 8 ? p[0] : p[0] + p[8];
  }
  return s;
}

constexpr int tp_red_floats(int T) { return kTpWaves * T * 16 * kTpRedCol; }
constexpr int tp_lds_bytes(int T) { return tp_red_floats(T) * 4; }

// Every sequence has left (EXIT mode)?
__device__ __forceinline__ bool tp_all_exited(const RowMap& rm, const WS& ws, const StepIO& io) {
  if (io.mode != EX_EXIT) return false;
  bool all = true;
  for (int sq = 0; sq < rm.nseq; ++sq) all &= ws.exited[sq] != 0;
  return all;
}

// ---- q, k, v (+ adapter-down rows when a fast row needs them) --------------------
template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_qkv(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io, int layer,
                                                        int fast_rows) {
  constexpr int T = kTpTiles;
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float ssum[kMaxRows * 4];
  __shared__ int ex_in[kMaxSeq], eb_in[kMaxSeq];
  __shared__ int reinit_s[kMaxSeq], exited_s[kMaxSeq], exitb_s[kMaxSeq];
  __shared__ float sig_s[kMaxSeq], asig_s[kMaxSeq];
  __shared__ float inv_rms[kMaxRows];
  __shared__ int take_s[kMaxRows];
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  const int th = D.th_qkv, nq = D.qdim, tq = nq / th;
  const int nqkv = 3 * nq + 3 * D.r;
  const int ntiles = 3 * tq + (fast_rows ? (3 * D.r + th - 1) / th : 0);
  if ((int)blockIdx.x >= ntiles) return;
  const size_t tb = (size_t)th * D.d * 2;
  const char* bq = (const char*)L.pq;   // q, k, v and the adapter-down rows are consecutive
  auto ptr = [&](int i) { return bq + (size_t)(blockIdx.x + i * gridDim.x) * tb; };
  const int n_local = (ntiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  TpCore<NS, MT, T> tc;
  tc.init(D.d, th, th * 64, ws.XB);
  // ---- requested before the weights: what the gate decision reads ----
  float bv[kBins];
  {
    const int q = min((int)threadIdx.x, rm.M * 4 - 1);
#pragma unroll
    for (int b = 0; b < kBins; ++b) bv[b] = bin_d_at(ws, layer, b, q >> 2)[q & 3];
  }
  const int sq0 = min((int)threadIdx.x, rm.nseq - 1);
  const int exv = ws.exited[sq0], ebv = ws.exitb[sq0];
  const float asv = (io.arla_sig ? io.arla_sig : ws.arla_sig)[sq0];
  __builtin_amdgcn_sched_barrier(0);
  tc.begin_w(ptr);
  sk_rm_copy(rmu, rm);
  if (threadIdx.x < rm.M * 4) {
    float s = 0.f;
#pragma unroll
    for (int b = 0; b < kBins; ++b) s += bv[b];
    ssum[threadIdx.x] = s;
  }
  if (threadIdx.x < rm.nseq) {
    ex_in[threadIdx.x] = exv;
    eb_in[threadIdx.x] = ebv;
    asig_s[threadIdx.x] = asv;
  }
  __syncthreads();
  if (threadIdx.x < rm.nseq)
    gate_logic(D, rml, ex_in, eb_in, io, layer, ssum, asig_s, reinit_s, exited_s, exitb_s, sig_s, threadIdx.x);
  __syncthreads();
  if (threadIdx.x < kMaxRows) {
    const int m = threadIdx.x;
    const bool take = m < rm.M && rml.fast[m] && reinit_s[rml.seq[m]] && rml.slow_of[m] >= 0;
    take_s[m] = take;   // (a fast row follows its slow row)
    inv_rms[m] = rsqrtf(ssum[min(take ? (int)rml.slow_of[m] : m, rm.M - 1) * 4] / D.d + D.eps);
  }
  if (blockIdx.x == 0 && threadIdx.x < rm.nseq) {
    const int sq = threadIdx.x;
    ws.reinit[layer * kMaxSeq + sq] = reinit_s[sq];
    ws.exited[sq] = exited_s[sq];
    ws.exitb[sq] = exitb_s[sq];
    if (layer > 0) ws.sig[sq * D.n_layers + layer - 1] = sig_s[sq];
  }
  __syncthreads();
  tc.begin_x(n_local, ptr, take_s[threadIdx.x & (MT > 8 ? 15 : 7)] != 0);
  tc.run(n_local, ptr, red, [&](int base, int cnt) {
    const int per = rm.M * th;
    for (int e = threadIdx.x; e < cnt * per; e += kTpThreads) {
      const int t = e / per, m = (e % per) / th, n = e % th;
      const int nn = (blockIdx.x + (base + t) * gridDim.x) * th + n;
      if (nn < nqkv) ws.QKV[(size_t)m * nqkv + nn] = tp_sum<MT, T>(red, t, m, n) * inv_rms[m];
    }
  });
}

// ---- o projection, residual add; sums for gate/up ---------------------------------
// One tile per workgroup where th * CUs covers d.
template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_oproj(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io, int layer,
                                                          int nf) {
  constexpr int T = 1;
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float uo_s[kMaxRows * kMaxRank];
  __shared__ float up_s[kTpThreads];
  __shared__ float newx[kMaxRows * 16];
  __shared__ float bo_s[kMaxRank * 16];       // first tile: B_o [j][row]
  __shared__ float agu_s[16 * 2 * kMaxRank];  // first tile: A_g, A_u times g_mlp [column][2 r]
  __shared__ float gm_s[16];                  // first tile: g_mlp
  __shared__ int flag_s[2 * kMaxSeq];         // exited, reinit
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  const int th = D.th_o, r = D.r;
  const int ntiles = (D.d + th - 1) / th;
  if ((int)blockIdx.x >= ntiles || tp_all_exited(rm, ws, io)) return;
  const size_t tb = (size_t)th * D.qdim * 2;
  auto ptr = [&](int i) { return (const char*)L.po + (size_t)(blockIdx.x + i * gridDim.x) * tb; };
  const int n_local = (ntiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  const int tid = threadIdx.x, n00 = blockIdx.x * th;
  const bool any_fast = nf > 0;
  TpCore<NS, MT, T> tc;
  tc.init(D.qdim, th, th * 64, ws.OB);
  // ---- requested before the weights: the first tile's epilogue operands
  // (unconditional loads at clamped indices) ----
  constexpr int NAG = 2 * kMaxRank * 16 / kTpThreads;   // A_g / A_u values per thread
  const int em = min(tid / th, rm.M - 1), en = tid % th;
  float xo = ws.X[(size_t)em * D.d + n00 + en];
  uint32_t braw = 0, araw[NAG] = {};
  float ag[NAG] = {};
  // o-adapter sums over the heads, of the fast rows (row 2k + 1 of a dual batch):
  // the threads share the heads of a (row, j) pair, 8 per thread and pass
  constexpr int UH = 8;
  float uo[UH] = {};
  const int items = nf * r, G = nf ? kTpThreads / items : 1;   // (at most 8 * 32 pairs)
  const int hpg = (D.H + G - 1) / G;
  const int ug = nf ? tid / items : 0, ui = nf ? tid - ug * items : 0;
  const float* up = ws.uo + ((size_t)(2 * (ui / max(r, 1)) + 1) * D.H) * r + ui % r;
  const int uh0 = min(ug * hpg, D.H), uh1 = ug < G ? min(uh0 + hpg, D.H) : uh0;
  float usum = 0.f;
  if (nf) {
#pragma unroll
    for (int u = 0; u < UH; ++u) uo[u] = up[(size_t)min(uh0 + u, D.H - 1) * r];
    const int bq = min(tid, th * r - 1);
    braw = ld_raw<1>(L.B[3] ? L.B[3] : L.po, (size_t)(n00 + bq / r) * r + bq % r);
#pragma unroll
    for (int k = 0; k < NAG; ++k) {
      const int aq = min(tid + k * kTpThreads, 2 * r * th - 1);
      const int which = aq / (r * th), j = (aq / th) % r, i = aq % th;
      const void* A = which ? L.A[5] : L.A[4];
      araw[k] = ld_raw<1>(A ? A : L.po, (size_t)j * D.d + n00 + i);
      ag[k] = L.mlp_norm[n00 + i];
    }
  }
  const float gm = L.mlp_norm[n00 + min(tid, th - 1)];
  const int fq = min(tid, 2 * rm.nseq - 1);
  const int fl = fq < rm.nseq ? ws.exited[fq] : ws.reinit[layer * kMaxSeq + fq - rm.nseq];
  __builtin_amdgcn_sched_barrier(0);
  tc.begin(n_local, ptr);
  sk_rm_copy(rmu, rm);
  if (tid < 2 * rm.nseq) flag_s[tid] = fl;
  if (tid < th) gm_s[tid] = gm;
  if (any_fast) {
#pragma unroll
    for (int u = 0; u < UH; ++u) usum += uh0 + u < uh1 ? uo[u] : 0.f;
    for (int h = uh0 + UH; h < uh1; ++h) usum += up[(size_t)h * r];
    up_s[tid] = usum;
    if (tid < th * r) bo_s[tid % r * 16 + tid / r] = L.B[3] ? raw_f<1>(braw) : 0.f;
#pragma unroll
    for (int k = 0; k < NAG; ++k) {
      const int q = tid + k * kTpThreads;
      if (q < 2 * r * th) {
        const void* A = q / (r * th) ? L.A[5] : L.A[4];
        agu_s[q % th * 2 * r + q / th] = A ? raw_f<1>(araw[k]) * ag[k] : 0.f;
      }
    }
    __syncthreads();
    if (tid < items) {
      float a = 0.f;
      for (int k = 0; k < G; ++k) a += up_s[k * items + tid];
      uo_s[(2 * (tid / r) + 1) * r + tid % r] = L.A[3] ? a : 0.f;   // (read after run's barrier)
    }
  }
  tc.run(n_local, ptr, red, [&](int base, int) {
    const bool first = base == 0;
    const int n0 = (blockIdx.x + base * gridDim.x) * th;
    const bool act = tid < rm.M * th;
    const int m = em, nn = n0 + en;
    float xnew = 0.f, pin = 0.f;
    bool upd = false;
    if (act) {
      const int sq = rml.seq[m];
      if (!first) xo = ws.X[(size_t)m * D.d + nn];
      xnew = xo;
      if (!flag_s[sq]) {
        upd = true;
        const float y = tp_sum<MT, T>(red, 0, m, en);
        if (rml.fast[m]) {
          // a fast row restarting at a gate takes its slow row's old value
          // (read here, before the barrier; written after it)
          pin = flag_s[rm.nseq + sq] ? ws.X[(size_t)rml.slow_of[m] * D.d + nn] : xo;
          float ad = 0.f;
          if (L.B[3] && L.A[3]) {
            if (first) {
#pragma unroll 8
              for (int j = 0; j < r; ++j) ad += bo_s[j * 16 + en] * uo_s[m * r + j];
            } else {
              ad = dot_row_t<1>(L.B[3], nn, r, uo_s + m * r);
            }
          }
          xnew = pin + y + ad;
        } else {
          xnew = xo + y;
        }
      }
      newx[m * 16 + en] = xnew;
    }
    __syncthreads();
    if (act) {
      if (upd) {
        ws.X[(size_t)m * D.d + nn] = xnew;
        if (rml.fast[m]) ws.PIN[(size_t)m * D.d + nn] = pin;
      }
      tp_put(ws.XB, m, nn, xnew * (first ? gm_s[en] : L.mlp_norm[nn]));
    }
    // sums for gate/up: x^2 of every row, and A_g, A_u times the fast rows over this tile's columns
    const int bin = blockIdx.x % kBins;
    for (int q = tid; q < rm.M + nf * 2 * r; q += kTpThreads) {
      const int f = q - rm.M;
      const int mm = f < 0 ? q : 2 * (f / (2 * r)) + 1, c = f < 0 ? 0 : f % (2 * r);
      const float* xm = newx + mm * 16;
      float v = 0.f;
      if (f < 0) {
#pragma unroll 4
        for (int i = 0; i < th; ++i) v += xm[i] * xm[i];
      } else if (first) {
#pragma unroll 4
        for (int i = 0; i < th; ++i) v += agu_s[i * 2 * r + c] * xm[i];
      } else {
        const void* A = c < r ? L.A[4] : L.A[5];
        if (A)
          for (int i = 0; i < th; ++i)
            v += ld_wt<1>(A, (size_t)(c % r) * D.d + n0 + i) * L.mlp_norm[n0 + i] * xm[i];
      }
      add_agent(bin_o_at(ws, D, layer, bin, mm) + (f < 0 ? 0 : 1 + c), v);
    }
  });
}

// ---- gate and up (pairs of tiles), SwiGLU; sums of the down adapter -----------------
template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_gateup(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io, int layer,
                                                           int nf) {
  constexpr int T = kTpTiles, NPAIR = T / 2;
  constexpr int NSV = (MT + MT * kMaxRank + kTpThreads - 1) / kTpThreads;   // sums per thread (half the rows are fast)
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float stat[kMaxRows * (1 + 2 * kMaxRank)];
  __shared__ float inv_rms[kMaxRows];
  __shared__ float act[NPAIR * kMaxRows * 16];
  // first group, raw: B_g, B_u [pair][which][j][16 rows], A_d [pair][j][16 columns], padded against bank conflicts
  __shared__ uint32_t bgu_s[NPAIR * 2 * kMaxRank * 17];
  __shared__ uint32_t ad_s[NPAIR * kMaxRank * 17];
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  const int r = D.r, ntiles = D.F / 16;
  if ((int)blockIdx.x >= ntiles || tp_all_exited(rm, ws, io)) return;
  const size_t tb = (size_t)16 * D.d * 2;
  // local tiles 2i, 2i+1: gate and up rows of pair blockIdx.x + i * gridDim.x, whose step blocks alternate
  auto ptr = [&](int i) {
    return (const char*)L.pg + (size_t)(blockIdx.x + (i >> 1) * gridDim.x) * 2 * tb + (i & 1) * 1024;
  };
  const int n_local = 2 * ((ntiles - blockIdx.x + gridDim.x - 1) / gridDim.x);
  const int PO = 1 + 2 * r, tid = threadIdx.x;
  const bool any_fast = nf > 0;
  // the sums read: x^2 of every row, the adapter sums of the fast rows (row 2k + 1 of a dual batch)
  const int nsum = rm.M + nf * 2 * r;
  auto sum_at = [&](int q, int& m, int& c) {
    const int f = max(q - rm.M, 0);
    m = q < rm.M ? q : 2 * (f / (2 * r)) + 1;
    c = q < rm.M ? 0 : 1 + f % (2 * r);
  };
  TpCore<NS, MT, T> tc;
  tc.init(D.d, 16, 2048, ws.XB);
  float sv[NSV][kBins];
#pragma unroll
  for (int k = 0; k < NSV; ++k) {
    if (k > 0 && k * kTpThreads >= nsum) break;   // (uniform)
    int m, c;
    sum_at(min(tid + k * kTpThreads, nsum - 1), m, c);
#pragma unroll
    for (int b = 0; b < kBins; ++b) sv[k][b] = bin_o_at(ws, D, layer, b, m)[c];
  }
  // the first group's B_g, B_u rows and A_d columns
  constexpr int NB = NPAIR * 2 * 16 * kMaxRank / kTpThreads, NAD = NPAIR * kMaxRank * 16 / kTpThreads;
  const int npair0 = min(NPAIR, n_local / 2);
  uint32_t pb[NB] = {}, pa[NAD] = {};
  if (any_fast) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      if (k * kTpThreads >= npair0 * 32 * r) break;
      const int q = min(tid + k * kTpThreads, npair0 * 32 * r - 1);
      const int p = q / (32 * r), which = (q / (16 * r)) & 1, rr = (q / r) % 16, j = q % r;   // (rows of B contiguous)
      const void* B = which ? L.B[5] : L.B[4];
      pb[k] = ld_raw<1>(B ? B : L.pg, (size_t)((blockIdx.x + p * gridDim.x) * 16 + rr) * r + j);
    }
#pragma unroll
    for (int k = 0; k < NAD; ++k) {
      if (k * kTpThreads >= npair0 * 16 * r) break;
      const int q = min(tid + k * kTpThreads, npair0 * 16 * r - 1);
      const int p = q / (16 * r), j = (q / 16) % r, i = q % 16;
      pa[k] = ld_raw<1>(L.A[6] ? L.A[6] : L.pg, (size_t)j * D.F + (blockIdx.x + p * gridDim.x) * 16 + i);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  tc.begin(n_local, ptr);
  sk_rm_copy(rmu, rm);
#pragma unroll
  for (int k = 0; k < NSV; ++k) {
    const int q = tid + k * kTpThreads;
    if (q >= nsum) break;
    float s = 0.f;
#pragma unroll
    for (int b = 0; b < kBins; ++b) s += sv[k][b];
    int m, c;
    sum_at(q, m, c);
    stat[m * PO + c] = s;
  }
  if (any_fast) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int q = tid + k * kTpThreads;
      if (q < npair0 * 32 * r) bgu_s[(q / (16 * r) * r + q % r) * 17 + (q / r) % 16] = pb[k];   // [p][which][j][n]
    }
#pragma unroll
    for (int k = 0; k < NAD; ++k) {
      const int q = tid + k * kTpThreads;
      if (q < npair0 * 16 * r) ad_s[q / 16 * 17 + q % 16] = pa[k];
    }
  }
  __syncthreads();
  if (tid < rm.M) inv_rms[tid] = rsqrtf(stat[tid * PO] / D.d + D.eps);   // (read after run's barrier)
  const bool hg = L.B[4] && L.A[4], hu = L.B[5] && L.A[5];
  tc.run(n_local, ptr, red, [&](int base, int cnt) {
    const bool first = base == 0;
    const int per = rm.M * 16, np = cnt / 2;
    for (int e = tid; e < np * per; e += kTpThreads) {
      const int p = e / per, m = (e % per) >> 4, n = e & 15;
      const int nn = (blockIdx.x + (base / 2 + p) * gridDim.x) * 16 + n;
      float g = tp_sum<MT, T>(red, 2 * p, m, n), u = tp_sum<MT, T>(red, 2 * p + 1, m, n);
      const float ir = inv_rms[m];
      if (rml.fast[m]) {
        const float* sg = stat + m * PO + 1;
        float dg = 0.f, du = 0.f;
        if (first) {
          const uint32_t* b = bgu_s + p * 2 * r * 17 + n;
#pragma unroll 8
          for (int j = 0; j < r; ++j) {
            dg += raw_f<1>(b[j * 17]) * sg[j];
            du += raw_f<1>(b[(r + j) * 17]) * sg[r + j];
          }
          if (!hg) dg = 0.f;
          if (!hu) du = 0.f;
        } else {
          if (hg) dg = dot_row_t<1>(L.B[4], nn, r, sg);
          if (hu) du = dot_row_t<1>(L.B[5], nn, r, sg + r);
        }
        g += dg;
        u += du;
      }
      const float av = silu(g * ir) * (u * ir);
      tp_put(ws.AB, m, nn, av);
      act[(p * kMaxRows + m) * 16 + n] = av;
    }
    if (!any_fast || !L.A[6]) return;   // (uniform)
    __syncthreads();
    // sums of the down adapter's down-projection over these columns: four lanes
    // per (fast row, j), a quarter of each tile's columns each
    const int bin = blockIdx.x % kBins;
    for (int q = tid; q < ((nf * r * 4 + 63) & ~63); q += kTpThreads) {
      const bool live = q < nf * r * 4;
      const int it = live ? q >> 2 : 0, mm = 2 * (it / r) + 1, j = it % r, i0 = (q & 3) * 4;
      float v = 0.f;
      for (int p = 0; p < np; ++p) {
        const float* a = act + (p * kMaxRows + mm) * 16 + i0;
        const size_t col = (size_t)j * D.F + (blockIdx.x + (base / 2 + p) * gridDim.x) * 16 + i0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          v += (first ? raw_f<1>(ad_s[(p * r + j) * 17 + i0 + i]) : ld_wt<1>(L.A[6], col + i)) * a[i];
      }
      v = quad_sum(v);
      if (live && (q & 3) == 0) add_agent(bin_gu_at(ws, D, layer, bin, mm) + j, v);
    }
  });
}

// ---- down projection, residual add; sums for the next norm and the exit signal -------
template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_down(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io, int layer,
                                                         const float* next_gain) {
  constexpr int T = 1;
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float ud[kMaxRows * kMaxRank];
  __shared__ float newx[kMaxRows * 16], pin_s[kMaxRows * 16];
  __shared__ float bd_s[kMaxRank * 16];   // first tile: B_d [j][row]
  __shared__ int ex_s[kMaxSeq];
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  const int th = D.th_d, r = D.r;
  const int ntiles = (D.d + th - 1) / th;
  if ((int)blockIdx.x >= ntiles) return;
  const bool idle = tp_all_exited(rm, ws, io);   // rows unchanged: planes and sums for the next layer only
  const size_t tb = (size_t)th * D.F * 2;
  auto ptr = [&](int i) { return (const char*)L.pd + (size_t)(blockIdx.x + i * gridDim.x) * tb; };
  const int n_local = (ntiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  const int tid = threadIdx.x, n00 = blockIdx.x * th;
  bool any_fast = false;
#pragma unroll
  for (int m = 0; m < kMaxRows; ++m) any_fast |= m < rm.M && rm.fast[m];
  const bool ad = any_fast && L.B[6] && L.A[6];
  TpCore<NS, MT, T> tc;
  tc.init(D.F, th, th * 64, ws.AB);
  float uv[kBins] = {};
  uint32_t pb = 0;
  if (ad) {
    const int q = min(tid, rm.M * r - 1);
#pragma unroll
    for (int b = 0; b < kBins; ++b) uv[b] = bin_gu_at(ws, D, layer, b, q / r)[q % r];
    const int bq = min(tid, th * r - 1);
    pb = ld_raw<1>(L.B[6], (size_t)(n00 + bq / r) * r + bq % r);
  }
  const int em = min(tid / th, rm.M - 1), en = tid % th;
  float x = ws.X[(size_t)em * D.d + n00 + en];
  float pi = ws.PIN[(size_t)em * D.d + n00 + en];
  float gn = next_gain[n00 + en];
  const int pe = ws.exited[min(tid, rm.nseq - 1)];
  __builtin_amdgcn_sched_barrier(0);
  if (!idle) tc.begin(n_local, ptr);
  sk_rm_copy(rmu, rm);
  if (ad && tid < rm.M * r) {
    float a = 0.f;
#pragma unroll
    for (int b = 0; b < kBins; ++b) a += uv[b];
    ud[tid] = a;
  }
  if (ad && tid < th * r) bd_s[tid % r * 16 + tid / r] = raw_f<1>(pb);
  if (tid < rm.nseq) ex_s[tid] = pe;
  auto epi = [&](int base, int) {
    const bool first = base == 0;
    const int n0 = (blockIdx.x + base * gridDim.x) * th, nn = n0 + en, m = em;
    if (tid < rm.M * th) {
      if (!first) {
        x = ws.X[(size_t)m * D.d + nn];
        pi = ws.PIN[(size_t)m * D.d + nn];
        gn = next_gain[nn];
      }
      if (!idle && !ex_s[rml.seq[m]]) {
        x += tp_sum<MT, T>(red, 0, m, en);
        if (ad && rml.fast[m]) {
          float a = 0.f;
          if (first) {
#pragma unroll 8
            for (int j = 0; j < r; ++j) a += bd_s[j * 16 + en] * ud[m * r + j];
          } else {
            a = dot_row_t<1>(L.B[6], nn, r, ud + m * r);
          }
          x += a;
        }
        ws.X[(size_t)m * D.d + nn] = x;
      }
      tp_put(ws.XB, m, nn, x * gn);
      newx[m * 16 + en] = x;
      pin_s[m * 16 + en] = rml.fast[m] ? pi : 0.f;
    }
    __syncthreads();
    const int bin = blockIdx.x % kBins;
    for (int q = tid; q < rm.M * 3; q += kTpThreads) {
      const int mm = q / 3, c = q % 3;
      if (c > 0 && !rml.fast[mm]) continue;
      float v = 0.f;
#pragma unroll 4
      for (int i = 0; i < th; ++i) {
        const float a = newx[mm * 16 + i], p = pin_s[mm * 16 + i];
        v += c == 0 ? a * a : (c == 1 ? p * a : p * p);
      }
      add_agent(bin_d_at(ws, layer + 1, bin, mm) + c, v);
    }
  };
  if (idle) {
    __syncthreads();
    for (int i = 0; i < n_local; ++i) {
      if (i) __syncthreads();
      epi(i, 1);
    }
    return;
  }
  tc.run(n_local, ptr, red, epi);
}

// The same with the reduction split over four workgroups (9 to 16 rows, long
// reductions).  With one workgroup per tile the planes of 16 rows are 2.7 times
// the weights' bytes through the L1; here a workgroup reads a quarter of them,
// for four tiles, and keeps them in registers.  The four leave partial sums in
// scratch; the last to arrive adds them in order and does the epilogue.  A
// reduction quarter stays on two of the eight XCDs (workgroup b % 8).
// d 3072, F 8192, 16 rows against one workgroup per tile: 20.4 -> 17.9 us
// (slow rows), 23.1 -> 20.2 us (eight dual sequences).
constexpr int kTpDownSplit = 4;
constexpr int kTpDownPart = kTpTiles * kMaxRows * 16;   // floats of one workgroup's partial sums

template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_down_split(Dims D, LayerPtrs L, RowMap rm, WS ws, StepIO io,
                                                               int layer, const float* next_gain, float* part) {
  constexpr int T = kTpTiles;
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float ud[kMaxRows * kMaxRank];
  __shared__ float newx[T * kMaxRows * 16], pin_s[T * kMaxRows * 16];
  __shared__ float bd_s[kMaxRank][T * 16 + 1];   // B_d [j][tile and row]
  __shared__ int ex_s[kMaxSeq];
  __shared__ int last_flag;
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  const int th = D.th_d, r = D.r, tid = threadIdx.x;
  const int ntiles = (D.d + th - 1) / th;
  const int x8 = blockIdx.x & 7, split = x8 >> 1, g = (int)(blockIdx.x >> 3) * 2 + (x8 & 1);
  const int n_local = min(T, ntiles - g * T);
  if (n_local <= 0) return;
  const bool idle = tp_all_exited(rm, ws, io);   // rows unchanged: planes and sums for the next layer only
  if (idle && split) return;
  const size_t tb = (size_t)th * D.F * 2;
  auto ptr = [&](int i) { return (const char*)L.pd + (size_t)(g * T + i) * tb; };
  bool any_fast = false;
#pragma unroll
  for (int m = 0; m < kMaxRows; ++m) any_fast |= m < rm.M && rm.fast[m];
  const bool ad = any_fast && L.B[6] && L.A[6];
  TpCore<NS, MT, T> tc;
  tc.init(D.F, th, th * 64, ws.AB, split, kTpDownSplit);
  float uv[kBins] = {};
  if (ad) {
    const int q = min(tid, rm.M * r - 1);
#pragma unroll
    for (int b = 0; b < kBins; ++b) uv[b] = bin_gu_at(ws, D, layer, b, q / r)[q % r];
  }
  // what the epilogue of the last to arrive reads, requested by all four before
  // the weights (16 dual rows: 23.1 us with these read after the arrival)
  const int per = rm.M * th, n = n_local * per, n0 = g * T * th;
  static_assert(T * kMaxRows * 16 == 2 * kTpThreads);
  float xv[2], pv[2], gv[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = min(tid + k * kTpThreads, n - 1), m = e % per / th, nn = n0 + e / per * th + e % th;
    xv[k] = ws.X[(size_t)m * D.d + nn];
    pv[k] = ws.PIN[(size_t)m * D.d + nn];
    gv[k] = next_gain[nn];
  }
  constexpr int NB = T * 16 * kMaxRank / kTpThreads;
  const int nb = n_local * th * r;
  uint32_t pb[NB] = {};
  if (ad) {
#pragma unroll
    for (int k = 0; k < NB; ++k) pb[k] = ld_raw<1>(L.B[6], (size_t)n0 * r + min(tid + k * kTpThreads, nb - 1));
  }
  const int pe = ws.exited[min(tid, rm.nseq - 1)];
  __builtin_amdgcn_sched_barrier(0);
  if (!idle) tc.begin(n_local, ptr);
  sk_rm_copy(rmu, rm);
  if (ad && tid < rm.M * r) {
    float a = 0.f;
#pragma unroll
    for (int b = 0; b < kBins; ++b) a += uv[b];
    ud[tid] = a;
  }
  if (ad) {
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int q = tid + k * kTpThreads;
      if (q < nb) bd_s[q % r][q / r] = raw_f<1>(pb[k]);
    }
  }
  if (tid < rm.nseq) ex_s[tid] = pe;
  __syncthreads();
  float* mine = part + ((size_t)g * kTpDownSplit + split) * kTpDownPart;
  if (!idle) {
    tc.run(n_local, ptr, red, [&](int, int) {
      for (int e = tid; e < n; e += kTpThreads) st_agent(&mine[e], tp_sum<MT, T>(red, e / per, e % per / th, e % th));
    });
    if (!arrive_last(&ws.att_cnt[g], kTpDownSplit, &last_flag)) return;
  }
  const float* all = part + (size_t)g * kTpDownSplit * kTpDownPart;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = tid + k * kTpThreads, t = e / per, m = e % per / th, c = e % th, nn = n0 + t * th + c;
    if (e >= n) continue;
    float x = xv[k];
    if (!idle && !ex_s[rml.seq[m]]) {
      float y = 0.f;
#pragma unroll
      for (int s2 = 0; s2 < kTpDownSplit; ++s2) y += ld_agent(&all[(size_t)s2 * kTpDownPart + e]);
      x += y;
      if (ad && rml.fast[m]) {
        float a = 0.f;
#pragma unroll 8
        for (int j = 0; j < r; ++j) a += bd_s[j][t * th + c] * ud[m * r + j];
        x += a;
      }
      ws.X[(size_t)m * D.d + nn] = x;
    }
    tp_put(ws.XB, m, nn, x * gv[k]);
    newx[(t * kMaxRows + m) * 16 + c] = x;
    pin_s[(t * kMaxRows + m) * 16 + c] = rml.fast[m] ? pv[k] : 0.f;
  }
  __syncthreads();
  const int bin = g % kBins;
  static_assert(T == 4 && kMaxRows * 3 * T <= kTpThreads);   // four lanes per sum, one tile each
  const int q = tid / T, mm = min(q / 3, rm.M - 1), c = q % 3, t = tid % T;
  float v = 0.f;
  if (t < n_local) {
#pragma unroll 4
    for (int i = 0; i < th; ++i) {
      const float a = newx[(t * kMaxRows + mm) * 16 + i], p = pin_s[(t * kMaxRows + mm) * 16 + i];
      v += c == 0 ? a * a : (c == 1 ? p * a : p * p);
    }
  }
  v = quad_sum(v);
  if (t == 0 && q < rm.M * 3 && (c == 0 || rml.fast[mm])) add_agent(bin_d_at(ws, layer + 1, bin, mm) + c, v);
}

// ---- final norm, LM head, arg-max; the last workgroup finishes the step -----------------
template <int NS, int MT>
__global__ __launch_bounds__(kTpThreads, 2) void kt_head(Dims D, const void* lm_head, RowMap rm, WS ws, StepIO io,
                                                         KVPtrs kv, int n_tiles, int n_layers_run) {
  constexpr int T = kTpTiles;
  extern __shared__ __attribute__((aligned(16))) float red[];
  __shared__ float ssum[kMaxRows * 4];
  __shared__ int hrow[kMaxRows], ex_in[kMaxSeq];
  __shared__ float bz_s[T * kMaxRows];   // this workgroup's arg-max so far, per (tile of a group, head row)
  __shared__ int bi_s[T * kMaxRows];
  __shared__ float inv_rms[kMaxRows];
  __shared__ int last_flag;
  __shared__ SkRmLds rmu;
  const RowMap& rml = rmu.rm;
  if ((int)blockIdx.x >= n_tiles) return;
  const size_t tb = (size_t)16 * D.d * 2;
  auto ptr = [&](int i) { return (const char*)lm_head + (size_t)(blockIdx.x + i * gridDim.x) * tb; };
  const int n_local = (n_tiles - blockIdx.x + gridDim.x - 1) / gridDim.x;
  TpCore<NS, MT, T> tc;
  tc.init(D.d, 16, 1024, ws.XB);
  float bv[kBins];
  {
    const int q = min((int)threadIdx.x, rm.M * 4 - 1);
#pragma unroll
    for (int b = 0; b < kBins; ++b) bv[b] = bin_d_at(ws, n_layers_run, b, q >> 2)[q & 3];
  }
  const int exv = ws.exited[min((int)threadIdx.x, rm.nseq - 1)];
  const int wgs = min((int)gridDim.x, n_tiles);
  __builtin_amdgcn_sched_barrier(0);
  tc.begin(n_local, ptr);
  HeadStates hs;
  hs.load(D, rm, ws, io, wgs);
  __builtin_amdgcn_sched_barrier(0);
  sk_rm_copy(rmu, rm);
  if (threadIdx.x < T * kMaxRows) {
    bz_s[threadIdx.x] = -INFINITY;
    bi_s[threadIdx.x] = 0x7fffffff;
  }
  if (threadIdx.x < rm.M * 4) {
    float s = 0.f;
#pragma unroll
    for (int b = 0; b < kBins; ++b) s += bv[b];
    ssum[threadIdx.x] = s;
  }
  if (threadIdx.x < rm.nseq) ex_in[threadIdx.x] = exv;
  __syncthreads();
  // rows that emit a token: every row of a chunk, else one per sequence
  const int nh = rm.head_all ? rm.M : rm.nseq;
  if (threadIdx.x < nh) {
    int pick = threadIdx.x;
    if (!rm.head_all) {
      const int sq = threadIdx.x, f = rml.first[sq], l = f + rml.cnt[sq] - 1;
      pick = rml.fast[l] && (ex_in[sq] || rml.slow_of[l] < 0) ? l : f;
    }
    hrow[threadIdx.x] = pick;
    inv_rms[threadIdx.x] = rsqrtf(ssum[pick * 4] / D.d + D.eps);   // (read after run's barrier)
  }
  tc.run(n_local, ptr, red, [&](int base, int cnt) {
    for (int e = threadIdx.x; e < ((cnt * nh * 16 + 63) & ~63); e += kTpThreads) {
      const bool live = e < cnt * nh * 16;
      const int t = live ? e / (nh * 16) : 0, k = live ? (e >> 4) % nh : 0, n = e & 15;
      const int tile = blockIdx.x + (base + t) * gridDim.x, nn = tile * 16 + n;
      float z = tp_sum<MT, T>(red, t, hrow[k], n) * inv_rms[k];
      if (nn >= D.V) z = -INFINITY;
      else if (live && io.logits_out) io.logits_out[(size_t)k * D.V + nn] = z;
      int idx = nn;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const float z2 = __shfl_xor(z, o);
        const int i2 = __shfl_xor(idx, o);
        if (z2 > z || (z2 == z && i2 < idx)) { z = z2; idx = i2; }
      }
      // (the same thread for the same slot in every group; ids rise from group
      // to group, so a tie takes a new id only over the empty slot's: a row of
      // infinitely low logits has the lowest id, too)
      const float bz = bz_s[t * kMaxRows + k];
      if (live && n == 0 && (z > bz || (z == bz && idx < bi_s[t * kMaxRows + k]))) {
        bz_s[t * kMaxRows + k] = z;
        bi_s[t * kMaxRows + k] = idx;
      }
    }
  });
  hs.store(D, rm, ws, io);
  __syncthreads();
  if (threadIdx.x < nh) {
    float z = -INFINITY;
    int idx = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float z2 = bz_s[t * kMaxRows + threadIdx.x];
      const int i2 = bi_s[t * kMaxRows + threadIdx.x];
      if (z2 > z || (z2 == z && i2 < idx)) { z = z2; idx = i2; }
    }
    st_agent(&ws.lm_val[(size_t)blockIdx.x * kMaxRows + threadIdx.x], z);
    st_agent(&ws.lm_idx[(size_t)blockIdx.x * kMaxRows + threadIdx.x], idx);
  }
  if (!arrive_last(ws.lm_cnt, wgs, &last_flag)) return;
  head_finish<4>(D, rm, rml, ws, io, kv, wgs, nh, ssum, false);
}

}  // namespace m2r2
