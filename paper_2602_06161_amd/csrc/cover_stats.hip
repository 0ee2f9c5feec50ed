// Producers of the seed-selection signals on gfx950 (arXiv 2602.06161, Sec. 5.3; Sec. 3).
//
// cover_token_stats_kernel: per row of the model's output logits, the log-probability of the
// token currently placed there (u = -log p, Sec. 5.3), the maximum probability (the
// confidence of Sec. 3) and the token attaining it.  One workgroup of 1024 threads per row;
// each thread streams 16-byte chunks with four loads in flight and keeps an online (max, sum
// of exp) pair and the chunk where its max was last raised, merged across the workgroup; the
// index inside that chunk is found at the end, by one thread of each wave that holds the row's
// maximum.  The placed token and its logit are fetched at the start by scalar loads.  HBM bounds
// it: 256 rows of 126464 bf16 logits (65 MB) 13.3 us, 15.0 when every thread read its best chunk
// again (a line from memory each, a quarter of the logits' bytes); 512 rows, cold, 29.1 -> 25.4.
//
// cover_attn_stats_kernel + cover_attn_stats_reduce_kernel: the in/out attention masses of
// Sec. 5.3 over a response region [r0, r0+Lr), from the last layer's corrected weights
// w_qj = exp(scale q.K^(q)_j - lse_q) (the same leave-one-out rows the attention computes,
// normalised over the whole sequence by the forward pass's lse), averaged over query heads:
//   d_in(j)  = (1/Hq) sum_h sum_{q masked} w_qj,    d_out(j) = (1/Hq) sum_h sum_{i drafted} w_ji
// Only masked queries count in d_in and only drafted keys in d_out, so the kernel first lists
// both (ascending) and multiplies just those rows: d_in takes S = Q_masked K^T over 32-key
// tiles, d_out takes S^T = K_drafted Q^T over 32-query tiles, the listed rows being the A
// operand, so that each mass is a sum inside a lane.  The listed rows are gathered into LDS once
// per workgroup, up to 512 at a time, by global-to-LDS loads; a wave keeps its own tiles' keys
// and queries in registers.  One workgroup per (batch row, query head, group of tiles), about
// 256 in all; both masses of its positions are complete in it and go to a caller-provided
// workspace, and a second kernel averages them over heads; every sum runs in a fixed order, so
// the results do not depend on scheduling.  Measured (B8 H32, 512 positions, 256 masked, 15
// drafted): forming S and S^T over all rows and keys with a mask 89 us; listed rows read by every
// wave on its own 32; through LDS 28.9, of which 14 are the 67 MB of Q and K at the rate HBM is
// read here and 3.5 the second kernel.
#include <hip/hip_runtime.h>

#include <mutex>
#include <stdint.h>

#include "cover.h"
#include "cover_internal.h"

namespace cover {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 gu32x4;

constexpr int kTokThreads = 1024;
constexpr int kTokUnroll = 4;  // 16-byte loads in flight per thread (more measured slower)
constexpr float kLog2e = 1.44269504088896341f;
constexpr float kLn2 = 0.693147180559945309f;
constexpr float kFloor = -1.0e30f;  // the lowest reference of a row's sum of exponentials

struct TokParams {
  const char* logits;
  const int32_t* tokens;
  float* logp;
  float* conf;
  int32_t* argmax;
  int64_t row_stride_bytes;
  int V;
};

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// the N values of a 16-byte chunk
template <bool BF>
__device__ __forceinline__ void unpack(u32x4 v, float* x) {
  if constexpr (BF) {
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[2 * e] = bf_lo(v[e]); x[2 * e + 1] = bf_hi(v[e]); }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(v[e]);
  }
}

// Per thread: the chunks c = tid + 1024 k in increasing order.  A chunk whose maximum exceeds
// the running one raises it (rescaling the sum) and becomes the thread's best chunk; the
// index inside that chunk is found once at the end, so the common path tracks no indices:
// a max over the chunk, then one exp2 per element into the sum.
template <bool BF>
__global__ __launch_bounds__(kTokThreads) void cover_token_stats_kernel(const TokParams p) {
#pragma clang fp contract(off)  // (the references below are rounded once, where they are formed)
  constexpr int N = BF ? 8 : 4;  // elements per 16-byte chunk
  __shared__ float sm[kTokThreads / 64], ss[kTokThreads / 64];
  __shared__ int si;
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const char* row = p.logits + (int64_t)r * p.row_stride_bytes;
  auto chunk = [&](int c) __attribute__((always_inline)) {
    return *(gu32x4*)((__attribute__((address_space(1))) const char*)row + (int64_t)c * 16);
  };
  const int nfull = p.V / N;  // whole chunks; the last V % N elements come after
  // the placed token's logit, requested now (uniform: scalar loads, apart from the stream)
  float xy = __builtin_nanf("");
  if (p.logp) {
    const int y = p.tokens[r];
    if ((unsigned)y < (unsigned)p.V) {
      if constexpr (BF) {
        const uint32_t w = *(const uint32_t*)(row + ((int64_t)y * 2 & ~(int64_t)3));
        xy = (y & 1) ? bf_hi(w) : bf_lo(w);
      } else {
        xy = *(const float*)(row + (int64_t)y * 4);
      }
    }
  }
  // s sums exp2(x log2 e + nm) with nm = -m log2 e rounded once: every term, rescaling and merge
  // uses that same rounded reference, and its rounding is taken out of the row's sum at the end.
  // The reference stays at kFloor where only lower logits (-inf, or the type's lowest value, whose
  // product leaves fp32) have been seen: they add zeros.
  float m = -INFINITY, nm = -(kFloor * kLog2e), s = 0.0f;
  int cbest = -1;
  auto fold = [&](const float* x, int c) __attribute__((always_inline)) {
#pragma clang fp contract(off)
    float cm = x[0];
#pragma unroll
    for (int e = 1; e < N; ++e) cm = __builtin_fmaxf(cm, x[e]);
    const float mn = __builtin_fmaxf(m, cm);
    const float nn = -(__builtin_fmaxf(mn, kFloor) * kLog2e);
    s *= __builtin_amdgcn_exp2f(nn - nm);  // 1 unless the max was raised
    cbest = cm > m ? c : cbest;
    m = mn;
    nm = nn;
    float a[N / 2];
#pragma unroll
    for (int e = 0; e < N / 2; ++e)
      a[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * e], kLog2e, nm)) +
             __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * e + 1], kLog2e, nm));
    float t = a[0];
#pragma unroll
    for (int e = 1; e < N / 2; ++e) t += a[e];
    s += t;
  };
  // rounds in which every thread's chunks exist: no bounds tests
  constexpr int kRound = kTokThreads * kTokUnroll;
  int c0 = tid;
  for (; c0 - tid + kRound <= nfull; c0 += kRound) {
    u32x4 v[kTokUnroll];
#pragma unroll
    for (int u = 0; u < kTokUnroll; ++u) v[u] = chunk(c0 + u * kTokThreads);
#pragma unroll
    for (int u = 0; u < kTokUnroll; ++u) {
      float x[N];
      unpack<BF>(v[u], x);
      fold(x, c0 + u * kTokThreads);
    }
  }
  {  // the last, partial round
    u32x4 v[kTokUnroll];
#pragma unroll
    for (int u = 0; u < kTokUnroll; ++u) {
      const int c = c0 + u * kTokThreads;
      v[u] = c < nfull ? chunk(c) : (u32x4){};
    }
#pragma unroll
    for (int u = 0; u < kTokUnroll; ++u) {
      const int c = c0 + u * kTokThreads;
      if (c < nfull) {
        float x[N];
        unpack<BF>(v[u], x);
        fold(x, c);
      }
    }
  }
  // the tail: one element per thread, read at its own width (never past the row's end)
  int ibest = 0x7fffffff;  // index of the thread's maximum, unless it is in chunk cbest
  if (tid < p.V - nfull * N) {
    const int j = nfull * N + tid;
    const float xj = BF ? __uint_as_float((uint32_t)(*(const uint16_t*)(row + (int64_t)j * 2)) << 16)
                        : *(const float*)(row + (int64_t)j * 4);
    if (xj > m) {
      m = xj;
      ibest = j;
      cbest = -1;
    }
    const float nn = -(__builtin_fmaxf(m, kFloor) * kLog2e);
    s = (s == 0.0f ? 0.0f : s * __builtin_amdgcn_exp2f(nn - nm)) + __builtin_amdgcn_exp2f(__builtin_fmaf(xj, kLog2e, nn));
    nm = nn;
  }
  // The row's maximum first: then only the threads that hold it read their best chunk again (a
  // line from HBM each: when every thread did, that was a quarter of the logits' bytes), while
  // the sums, on the common maximum, are added.
  float wm = m;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) wm = __builtin_fmaxf(wm, __shfl_xor(wm, off));
  if (lane == 0) sm[wave] = wm;
  if (tid == 0) si = 0x7fffffff;
  __syncthreads();
  float M = sm[0];
#pragma unroll
  for (int w = 1; w < kTokThreads / 64; ++w) M = __builtin_fmaxf(M, sm[w]);
  // (of several threads of a wave, on rows with ties, only the one with the smallest index does:
  // their chunks don't overlap, and a tail element lies behind every chunk)
  bool holds = m == M;
  if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(holds)) > 1) {
    const int key = holds ? (cbest >= 0 ? cbest * N : ibest) : 0x7fffffff;
    int least = key;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) least = min(least, __shfl_xor(least, off));
    holds = key == least;
  }
  u32x4 best = {};
  if (holds && cbest >= 0) best = chunk(cbest);
  const bool plain = __builtin_fabsf(M) < -kFloor;
  float nM = -(M * kLog2e);
  float t = s == 0.0f ? 0.0f : s * __builtin_amdgcn_exp2f(nM - nm);
  if (!plain) {  // no logit above kFloor, or products beyond fp32: the sum again, by differences
    nM = t = 0.0f;
    for (int j = tid; j < p.V; j += kTokThreads) {
      const float xj = BF ? __uint_as_float((uint32_t)((const uint16_t*)row)[j] << 16) : ((const float*)row)[j];
      t += __builtin_amdgcn_exp2f((xj - M) * kLog2e);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
  if (lane == 0) ss[wave] = t;
  if (holds) {  // the first element of the best chunk that holds the maximum; ties: the smallest
    if (cbest >= 0) {
      float x[N];
      unpack<BF>(best, x);
#pragma unroll
      for (int e = N - 1; e >= 0; --e)
        if (x[e] == M) ibest = cbest * N + e;
    }
    atomicMin(&si, ibest);
  }
  __syncthreads();
  if (tid == 0) {
    float a[kTokThreads / 64];
#pragma unroll
    for (int w = 0; w < kTokThreads / 64; ++w) a[w] = ss[w];
#pragma unroll
    for (int n = kTokThreads / 128; n >= 1; n >>= 1)
#pragma unroll
      for (int w = 0; w < n; ++w) a[w] += a[w + n];
    // the sum is 2^c times that of exp(x - M), c the rounding of nM
    const float c = plain ? __builtin_fmaf(M, kLog2e, nM) : 0.0f;
    const float lz = __builtin_fmaf(__builtin_amdgcn_logf(a[0]) - c, kLn2, M);  // natural log-sum-exp
    if (p.conf) p.conf[r] = __builtin_amdgcn_exp2f(c) / a[0];        // exp(max - lz)
    if (p.argmax) p.argmax[r] = si < p.V ? si : 0;  // (no number in the row)
    if (p.logp) p.logp[r] = xy - lz;
  }
}


// ---------------------------------------------------------------------------------------
// attention masses
// ---------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct StatParams {
  const __bf16* q;
  const __bf16* kl;
  const __bf16* kc;
  const int32_t* seed_idx;
  const int32_t* n_seed;
  const float* lse;
  const uint8_t* masked;
  const uint8_t* drafted;
  float* ws;  // [B, Hq, 2, Lr]: per head, d_in and d_out
  float* d_in;
  float* d_out;
  int B, Hq, Hkv, L, d, max_seeds, group, r0, Lr, NB;
  int KG, TPG, wpk;  // workgroups per head, 32-position tiles per workgroup, waves per tile
  float scale;
  int64_t q_sb, q_sh, q_sl, kv_sb, kv_sh, kv_sl;
};

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// 16 values, in a tree of depth 4 (a chain of 16 rounds the larger partial sums 16 times)
__device__ __forceinline__ float tree_sum(const f32x4* w) {
  const f32x4 a = (w[0] + w[1]) + (w[2] + w[3]);
  return (a[0] + a[1]) + (a[2] + a[3]);
}

constexpr int kStatWaves = 8;
constexpr int kStatThreads = 64 * kStatWaves;
constexpr int kSegs = COVER_STATS_MAX_LR / 64;              // 64-position segments of the region
constexpr int kPos = COVER_STATS_MAX_LR / kStatThreads;     // region positions per thread
static_assert(kPos * kStatThreads == COVER_STATS_MAX_LR, "the region is dealt out evenly");

// NK: key tiles (and query tiles) a wave holds at a time, so that each gathered row feeds NK MFMAs
// DIRECT: the listed rows are read from memory by the wave that multiplies them (up to two tiles
// per workgroup, where a row is used once or twice and LDS would only add a round trip: B1 H32,
// 256 positions 8.9 us a call against 9.9); otherwise through LDS
template <int D, int NK, bool DIRECT>
__global__ __launch_bounds__(kStatThreads) void cover_attn_stats_kernel(const StatParams p) {
  constexpr int KS = D / 16;
  constexpr int kCap = D == 128 ? 16 : 14;  // units in LDS (D = 64: two workgroups per CU)
  __shared__ __attribute__((aligned(1024))) char rows[DIRECT ? 1024 : kCap * 32 * 2 * D];
  __shared__ uint64_t seg_m[kSegs], seg_d[kSegs];           // masked / drafted positions
  __shared__ uint32_t sbits[2 * kSegs];                     // seeds
  __shared__ uint16_t list_m[COVER_STATS_MAX_LR], list_d[COVER_STATS_MAX_LR];
  __shared__ __attribute__((aligned(16))) float lse_m[COVER_STATS_MAX_LR];  // of the masked queries
  __shared__ float part_in[kStatWaves][32], part_out[kStatWaves][32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hl = lane >> 5, l32 = lane & 31;
  const int kg = blockIdx.x % p.KG, bh = blockIdx.x / p.KG;
  const int h = bh % p.Hq, b = bh / p.Hq;
  const int kt0 = kg * p.TPG, kt1 = min(p.NB, kt0 + p.TPG);  // this workgroup's tiles of positions
  float* const wsh = p.ws + ((int64_t)b * p.Hq + h) * 2 * p.Lr;
  const int g = h / p.group;
  const int Lr = p.Lr;
  const __bf16* qbh = p.q + b * p.q_sb + h * p.q_sh + p.r0 * p.q_sl;  // region position 0
  const int64_t kvo = b * p.kv_sb + g * p.kv_sh + p.r0 * p.kv_sl;
  const float* lrow = p.lse + ((int64_t)b * p.Hq + h) * p.L + p.r0;
  // (the difference before the change of base: rounding lse log2 e first costs up to 2^-24 of
  // its size in every weight of a query)
  const float scale = p.scale;
  auto weight = [=](float s, float lse) __attribute__((always_inline)) -> float {
    return __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale, -lse) * kLog2e);
  };

  // ---- the seed count and list, membership and lse of every position: one round trip --------
  const int ns_raw = p.max_seeds > 0 ? p.n_seed[b] : 0;
  const int j_first = tid < p.max_seeds ? p.seed_idx[(int64_t)b * p.max_seeds + tid] : -1;
  uint8_t mb[kPos], db[kPos];
  float ls[kPos];
#pragma unroll
  for (int m = 0; m < kPos; ++m) {
    const int j = tid + m * kStatThreads;
    mb[m] = db[m] = 0;
    ls[m] = 0.0f;
    if (j < Lr) {
      mb[m] = p.masked[(int64_t)b * Lr + j];
      db[m] = p.drafted[(int64_t)b * Lr + j];
      ls[m] = lrow[j];
    }
  }
  if (tid < 2 * kSegs) sbits[tid] = 0u;
  __syncthreads();
  // seeds of the region, and the masked and drafted positions as ascending lists
  const int ns = ns_raw < 0 ? 0 : (ns_raw > p.max_seeds ? p.max_seeds : ns_raw);
  auto mark = [&](int j) {
    const int64_t t = (int64_t)j - p.r0;
    if (t >= 0 && t < Lr) atomicOr(&sbits[t >> 5], 1u << (t & 31));
  };
  if (tid < ns) mark(j_first);
  for (int t = tid + kStatThreads; t < ns; t += kStatThreads) mark(p.seed_idx[(int64_t)b * p.max_seeds + t]);
  const int n_seg = (Lr + 63) >> 6;
#pragma unroll
  for (int m = 0; m < kPos; ++m) {
    const uint64_t um = __builtin_amdgcn_ballot_w64(mb[m] != 0), ud = __builtin_amdgcn_ballot_w64(db[m] != 0);
    if (lane == 0) {
      seg_m[m * kStatWaves + wave] = um;
      seg_d[m * kStatWaves + wave] = ud;
    }
  }
  __syncthreads();
  int n_m = 0, n_d = 0, base_m[kPos], base_d[kPos];
  for (int s = 0; s < n_seg; ++s) {
#pragma unroll
    for (int m = 0; m < kPos; ++m)
      if (s == m * kStatWaves + wave) {
        base_m[m] = n_m;
        base_d[m] = n_d;
      }
    n_m += __builtin_popcountll(seg_m[s]);
    n_d += __builtin_popcountll(seg_d[s]);
  }
#pragma unroll
  for (int m = 0; m < kPos; ++m) {
    const int s = m * kStatWaves + wave;
    if (s < n_seg) {
      const uint64_t um = seg_m[s], ud = seg_d[s], below = (1ull << lane) - 1;
      if ((um >> lane) & 1) {
        const int at = base_m[m] + __builtin_popcountll(um & below);
        list_m[at] = (uint16_t)(s * 64 + lane);
        lse_m[at] = ls[m];
      }
      if ((ud >> lane) & 1) list_d[base_d[m] + __builtin_popcountll(ud & below)] = (uint16_t)(s * 64 + lane);
    }
  }
  // a last partial tile of masked queries: no weight
  const int m_tiles = (n_m + 31) >> 5, d_tiles = (n_d + 31) >> 5;
  if (tid < 32 * m_tiles - n_m) lse_m[n_m + tid] = INFINITY;
  __syncthreads();

  auto is_seed = [&](int j) -> bool { return (sbits[j >> 5] >> (j & 31)) & 1u; };
  auto load_q = [&](bf16x8* f, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = *(const bf16x8*)(qbh + (int64_t)j * p.q_sl + (2 * ks + hl) * 8);
  };
  auto k_row = [&](int j) __attribute__((always_inline)) -> const __bf16* {
    return (is_seed(j) ? p.kc : p.kl) + kvo + (int64_t)j * p.kv_sl;
  };
  auto load_k = [&](bf16x8* f, int j) __attribute__((always_inline)) {
    const __bf16* src = k_row(j);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = *(const bf16x8*)(src + (2 * ks + hl) * 8);
  };
  // The units: m_tiles tiles of listed masked queries, then d_tiles tiles of listed drafted keys.
  // Their rows are gathered into LDS, kCap units at a time, by global-to-LDS loads of kRPL rows
  // (lane / kCh selects the row, past the list's end its last entry), the 16-byte chunk index
  // XOR-ed with the row's swizzle, so that the b128 operand reads cover all banks.
  constexpr int kCh = D / 8, kRPL = 64 / kCh, kLPU = 32 / kRPL;  // loads per unit
  auto swz = [](int row) __attribute__((always_inline)) -> int { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  const int units = m_tiles + d_tiles;
  auto stage = [&](int u0) __attribute__((always_inline)) {
    const int n = min(units - u0, kCap) * kLPU;
    for (int i = wave; i < n; i += kStatWaves) {
      const int u = u0 + i / kLPU, r = (i % kLPU) * kRPL + lane / kCh;
      const __bf16* src;
      if (u < m_tiles) src = qbh + (int64_t)list_m[min(32 * u + r, n_m - 1)] * p.q_sl;
      else src = k_row(list_d[min(32 * (u - m_tiles) + r, n_d - 1)]);
      __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)(src + ((lane % kCh) ^ swz(r)) * 8),
                                       (__attribute__((address_space(3))) void*)(rows + i * 1024), 16, 0, 0);
    }
  };
  // q_j . k_live_j of this lane's position (both halves of d)
  auto live_score = [&](int j) -> float {
    const __bf16* qr = qbh + (int64_t)j * p.q_sl;
    const __bf16* kr = p.kl + kvo + (int64_t)j * p.kv_sl;
    float acc = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 qv = *(const bf16x8*)(qr + (2 * ks + hl) * 8), kv = *(const bf16x8*)(kr + (2 * ks + hl) * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = __builtin_fmaf((float)qv[e], (float)kv[e], acc);
    }
    return acc + __shfl_xor(acc, 32);
  };

  // ---- the masses of the workgroup's tiles --------------------------------------------------
  // With up to 4 tiles wpk waves share a tile's units (unit u: wave u % wpk of them) and the sums
  // are added in order below; otherwise a wave takes NK tiles at a time and all units.
  const int part = p.wpk > 1 ? wave % p.wpk : 0;
  const int n_iter = p.wpk > 1 ? 1 : (kt1 - kt0 + kStatWaves * NK - 1) / (kStatWaves * NK);
  for (int it = 0; it < n_iter; ++it) {
    const int kt = kt0 + (p.wpk > 1 ? wave / p.wpk : (it * kStatWaves + wave) * NK);
    const bool active = kt < kt1;
    if (!DIRECT && it == 0 && units > 0) stage(0);
    int jt[NK];            // this lane's position in each tile (clamped into the region)
    float din[NK], dout[NK], lq[NK];
    uint32_t own[NK];      // positions whose diagonal takes the live key: seed and masked or drafted
    float s_live[NK];
    uint32_t any_own = 0;
#pragma unroll
    for (int n = 0; n < NK; ++n) {
      const int t = min(kt + n, p.NB - 1);
      jt[n] = min(32 * t + l32, Lr - 1);
      din[n] = dout[n] = s_live[n] = lq[n] = 0.0f;
      const uint32_t half = 32 * (t & 1);
      own[n] = sbits[t] & ((uint32_t)(seg_m[t >> 1] >> half) | (uint32_t)(seg_d[t >> 1] >> half));
      any_own |= own[n];
    }
    // the tiles' rows as B operands: keys for the masked queries, queries for the drafted keys
    // (requested together, while the units are on their way to LDS)
    bf16x8 fk[NK][KS], fq[NK][KS];
    if (active && part < m_tiles) {
#pragma unroll
      for (int n = 0; n < NK; ++n) load_k(fk[n], jt[n]);
    }
    if (active && ((part - m_tiles) & (p.wpk - 1)) < d_tiles) {
#pragma unroll
      for (int n = 0; n < NK; ++n) {
        load_q(fq[n], jt[n]);
        lq[n] = lrow[jt[n]];
      }
    }
    if (__builtin_amdgcn_readfirstlane(any_own) != 0) {
#pragma unroll
      for (int n = 0; n < NK; ++n) s_live[n] = live_score(jt[n]);
    }
    // seed rows on their own diagonal: the listed position equals this lane's
    auto diagonal = [&](f32x16* s, const uint16_t* list, int n_list, int t) {
      const int lo = list[32 * t], hi = list[min(32 * t + 31, n_list - 1)];
#pragma unroll
      for (int n = 0; n < NK; ++n) {
        if (hi < 32 * (kt + n) || lo > 32 * (kt + n) + 31) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int at = 32 * t + 8 * (r >> 2) + 4 * hl + (r & 3);
          if (at < n_list && list[at] == 32 * (kt + n) + l32 && ((own[n] >> l32) & 1u)) s[n][r] = s_live[n];
        }
      }
    };
    for (int u0 = 0; u0 < units; u0 += DIRECT ? units : kCap) {
      const bool again = !DIRECT && (u0 > 0 || (it > 0 && units > kCap));
      if (again) {
        __syncthreads();  // (every wave is done with the units before)
        stage(u0);
      }
      if (!DIRECT && (again || it == 0)) {
        __builtin_amdgcn_s_waitcnt(0);  // this wave's loads to LDS have landed, so after
        __syncthreads();                // the barrier have all waves'
      }
      if (!active) continue;
      const int u1 = DIRECT ? units : min(units, u0 + kCap);
      for (int u = u0 + ((part - u0) & (p.wpk - 1)); u < u1; u += p.wpk) {
        // the listed rows (A) against the wave's tiles (B): S in the registers of (row, position)
        const char* base = rows + (u - u0) * (32 * 2 * D) + l32 * (2 * D);
        bf16x8 fa[KS];
        if constexpr (DIRECT) {
          if (u < m_tiles) load_q(fa, list_m[min(32 * u + l32, n_m - 1)]);
          else load_k(fa, list_d[min(32 * (u - m_tiles) + l32, n_d - 1)]);
        }
#pragma unroll
        for (int ks = 0; ks < KS && !DIRECT; ++ks) fa[ks] = *(const bf16x8*)(base + (((2 * ks + hl) ^ swz(l32)) << 4));
        f32x16 s[NK];
#pragma unroll
        for (int n = 0; n < NK; ++n) s[n] = (f32x16){};
        if (u < m_tiles) {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int n = 0; n < NK; ++n) s[n] = mfma16(fa[ks], fk[n][ks], s[n]);
          if (__builtin_amdgcn_readfirstlane(any_own) != 0) diagonal(s, list_m, n_m, u);
          f32x4 w4[NK][4];  // a unit's 16 weights are added as a tree, then to the running sum
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 lm = *(const f32x4*)(lse_m + 32 * u + 8 * q + 4 * hl);
#pragma unroll
            for (int n = 0; n < NK; ++n)
#pragma unroll
              for (int e = 0; e < 4; ++e) w4[n][q][e] = weight(s[n][4 * q + e], lm[e]);
          }
#pragma unroll
          for (int n = 0; n < NK; ++n) din[n] += tree_sum(w4[n]);
        } else {
          const int t = u - m_tiles;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int n = 0; n < NK; ++n) s[n] = mfma16(fa[ks], fq[n][ks], s[n]);
          if (__builtin_amdgcn_readfirstlane(any_own) != 0) diagonal(s, list_d, n_d, t);
          const int lim = n_d - 32 * t - 4 * hl;  // rows past the list's end have no weight
#pragma unroll
          for (int n = 0; n < NK; ++n) {
            f32x4 w4[4];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const float w = weight(s[n][r], lq[n]);
              w4[r >> 2][r & 3] = 8 * (r >> 2) + (r & 3) < lim ? w : 0.0f;
            }
            dout[n] += tree_sum(w4);
          }
        }
      }
    }
#pragma unroll
    for (int n = 0; n < NK; ++n) {
      din[n] += __shfl_xor(din[n], 32);
      dout[n] += __shfl_xor(dout[n], 32);
      if (p.wpk > 1) {  // (one tile per wave then: TPG <= kStatWaves / wpk)
        if (hl == 0 && active) {
          part_in[wave][l32] = din[n];
          part_out[wave][l32] = dout[n];
        }
      } else if (hl == 0 && kt + n < kt1 && 32 * (kt + n) + l32 < Lr) {
        wsh[32 * (kt + n) + l32] = din[n];
        wsh[Lr + 32 * (kt + n) + l32] = dout[n];
      }
    }
  }
  if (p.wpk > 1) {
    __syncthreads();
    const int t = kt0 + (tid >> 5);  // tile of this thread, position tid % 32
    if (t < kt1 && 32 * t + l32 < Lr) {
      float a = 0.0f, c = 0.0f;
      for (int w = 0; w < p.wpk; ++w) {
        a += part_in[(t - kt0) * p.wpk + w][l32];
        c += part_out[(t - kt0) * p.wpk + w][l32];
      }
      wsh[32 * t + l32] = a;
      wsh[Lr + 32 * t + l32] = c;
    }
  }
}

// d_in(j) = (1/Hq) sum_h ws[h][0][j], d_out(j) = (1/Hq) sum_h ws[h][1][j].  A block of 32
// keys x 8 head lanes: lane y adds heads y, y+8, ..., then the 8 lane sums are added in order:
// a fixed order, so deterministic.
__global__ __launch_bounds__(256) void cover_attn_stats_reduce_kernel(const StatParams p) {
  __shared__ float sin_[8][32], sout[8][32];
  const int b = blockIdx.y, jx = threadIdx.x & 31, hy = threadIdx.x >> 5;
  const int j = blockIdx.x * 32 + jx;
  float din = 0.0f, dout = 0.0f;
  if (j < p.Lr) {
    const float* w = p.ws + (int64_t)b * p.Hq * 2 * p.Lr + j;
#pragma unroll 4
    for (int h = hy; h < p.Hq; h += 8) {
      din += w[(int64_t)(2 * h) * p.Lr];
      dout += w[(int64_t)(2 * h + 1) * p.Lr];
    }
  }
  sin_[hy][jx] = din;
  sout[hy][jx] = dout;
  __syncthreads();
  if (hy == 0 && j < p.Lr) {
    float a = 0.0f, c = 0.0f;
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      a += sin_[y][jx];
      c += sout[y][jx];
    }
    const float inv = 1.0f / (float)p.Hq;
    p.d_in[(int64_t)b * p.Lr + j] = a * inv;
    p.d_out[(int64_t)b * p.Lr + j] = c * inv;
  }
}

}  // namespace

hipError_t launch_token_stats(const TokenArgs& a, hipStream_t stream) {
  TokParams p;
  p.logits = (const char*)a.logits;
  p.tokens = a.tokens;
  p.logp = a.logp;
  p.conf = a.conf;
  p.argmax = a.argmax;
  p.row_stride_bytes = a.row_stride * (a.bf16 ? 2 : 4);
  p.V = a.V;
  if (a.bf16)
    hipLaunchKernelGGL(cover_token_stats_kernel<true>, dim3((unsigned)a.R), dim3(kTokThreads), 0, stream, p);
  else
    hipLaunchKernelGGL(cover_token_stats_kernel<false>, dim3((unsigned)a.R), dim3(kTokThreads), 0, stream, p);
  return hipGetLastError();
}

// The workspace of cover_attn_stats_noalloc: one array per GPU, held until the process ends.
// Host code never passes `scratch` itself to a kernel (in host code the name stands for a
// host-side shadow, not a device address); it passes the address hipGetSymbolAddress gives
// for the current device.
static __device__ __align__(256) float scratch[COVER_STATS_SCRATCH_FLOATS];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t stats_scratch(float** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = (float*)p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

void stats_key_groups(int B, int Hq, int Lr, int* tpg, int* kg_out) {
  // key groups: about 256 workgroups in all (at most one group per 32-key tile, none empty)
  const int nb = (Lr + 31) / 32;
  const int64_t heads = (int64_t)B * Hq;
  int64_t kg = heads > 0 ? (256 + heads - 1) / heads : 1;
  kg = kg < 1 ? 1 : (kg > nb ? nb : kg);
  const int t = kg > 0 ? (int)((nb + kg - 1) / kg) : 1;
  *tpg = t;
  *kg_out = t > 0 ? (nb + t - 1) / t : 0;
}

int64_t stats_workspace_floats(int B, int Hq, int Lr) {
  int tpg, kg;
  stats_key_groups(B, Hq, Lr, &tpg, &kg);
  return (int64_t)B * Hq * (1 + kg) * Lr;
}

hipError_t launch_attn_stats(const StatsArgs& a, hipStream_t stream) {
  StatParams p;
  p.q = (const __bf16*)a.q;
  p.kl = (const __bf16*)a.k_live;
  p.kc = (const __bf16*)a.k_cache;
  p.seed_idx = a.seed_idx;
  p.n_seed = a.n_seed;
  p.lse = a.lse;
  p.masked = a.masked;
  p.drafted = a.drafted;
  p.ws = a.workspace;
  p.d_in = a.d_in;
  p.d_out = a.d_out;
  p.B = a.B; p.Hq = a.Hq; p.Hkv = a.Hkv; p.L = a.L; p.d = a.d; p.max_seeds = a.max_seeds;
  p.group = a.Hq / a.Hkv;
  p.r0 = a.r0; p.Lr = a.Lr;
  p.NB = (a.Lr + 31) / 32;
  stats_key_groups(a.B, a.Hq, a.Lr, &p.TPG, &p.KG);
  p.scale = a.scale;
  p.q_sb = a.q_sb; p.q_sh = a.q_sh; p.q_sl = a.q_sl;
  p.kv_sb = a.kv_sb; p.kv_sh = a.kv_sh; p.kv_sl = a.kv_sl;
  const int64_t nwg = (int64_t)a.B * a.Hq * p.KG;
  if (nwg > 0x7fffffff) return hipErrorInvalidConfiguration;
  // Up to 4 tiles per workgroup several waves share one; past 8 a wave holds two at a time, so
  // that every listed row feeds two products (32 us against 46 at B8 H32, 512 positions, when
  // rows came straight from memory).
  p.wpk = p.TPG <= 1 ? 8 : (p.TPG <= 2 ? 4 : (p.TPG <= 4 ? 2 : 1));
  const dim3 grid((unsigned)nwg), block(kStatThreads);
  if (a.d == 128) {
    if (p.TPG <= 2) hipLaunchKernelGGL((cover_attn_stats_kernel<128, 1, true>), grid, block, 0, stream, p);
    else if (p.TPG <= 8) hipLaunchKernelGGL((cover_attn_stats_kernel<128, 1, false>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((cover_attn_stats_kernel<128, 2, false>), grid, block, 0, stream, p);
  } else {
    if (p.TPG <= 2) hipLaunchKernelGGL((cover_attn_stats_kernel<64, 1, true>), grid, block, 0, stream, p);
    else if (p.TPG <= 8) hipLaunchKernelGGL((cover_attn_stats_kernel<64, 1, false>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((cover_attn_stats_kernel<64, 2, false>), grid, block, 0, stream, p);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cover_attn_stats_reduce_kernel, dim3((unsigned)((a.Lr + 31) / 32), (unsigned)a.B),
                     dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace cover
