// COVER attention on gfx950, fp32: bidirectional attention over the KV-cache-overridden memory
// with the diagonal correction for seed rows (arXiv 2602.06161, Sec. 5.1 and App. B).
//
// What every query row i of batch row b computes (S_b = seed set of b):
//   K'_j = k_cache_j if j in S_b else k_live_j          (override memory, Sec. 5.1)
//   row view: K'_j for j != i;  k_live_i at j == i when i in S_b   (leave-one-out view)
//   out_i = softmax_j(scale <q_i, K^(i)_j>) V^(i),  lse_i = log sum_j exp(...)
// The paper derives the seed-row result as a post-hoc rescaling of the overridden row
// (Lemma B.1, closed form of App. B.4).  Here the overridden diagonal gets no weight in the main
// loop and the live diagonal term joins the row's softmax at the end, so there is no division
// by r_i (by Lemma B.1 the two are equal in exact arithmetic; this form has no cancellation
// when the cached diagonal dominates the row).  The bf16 kernels are in cover_attn_w4.hip.
//
// On the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums).  One workgroup of up to 8 waves
// (one, where there are enough) per 16 query rows of one (b, h); the waves take the 16-key tiles in
// turn and merge their (max, sum, O) through LDS.  The calls are small (a layer of tens to hundreds of tokens), so
// what bounds them is latency: 16-row tiles give the most workgroups and the shortest chain per
// tile (1024 matrix cycles at d = 64), each wave requests its next tile before it works on one,
// and every operand is read from memory in the layout the instruction wants, without LDS:
//   S^T = K Q^T   lane (i, g) = (lane % 16, lane / 16) holds 4 consecutive d of key row i (of
//                 query row i), d = 16 s + 4 g + e; product (s, e) takes element e of both, so
//                 the order of d is the same on both sides
//   O^T = V^T P^T the S^T registers of lane (i, g) are keys 4 g + r of query i: the B operand
//                 of product r.  A: 4 consecutive d of key row 4 g + r, d = 64 c + 4 i + e;
//                 accumulator (c, e) then holds O at d = 64 c + 4 row + e
// Measured against one lane per query row walking the keys: B1 H2 L64 d64 51.2 -> 4.9 us,
// B2 H8 L640 d64 464 -> 40, B1 H32 L1024 d128 2040 -> 251 (69 of the instruction's 157 TFLOP/s;
// placing a head's workgroups on one XCD changed nothing, so it is not L2 misses that bound it).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cover.h"
#include "cover_internal.h"

namespace cover {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kInitMax = -1.0e30f; // finite "no key seen yet" reference max
constexpr float kLn2 = 0.693147180559945309f;

__device__ __forceinline__ float swap_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float swap_add(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fmax2(float a, float b) { return __builtin_fmaxf(a, b); }

struct ParamsF {
  const float* q;
  const float* kl;
  const float* vl;
  const float* kc;
  const float* vc;
  const int32_t* seed_idx;
  const int32_t* n_seed;
  float* out;
  float* lse;
  int B, Hq, Hkv, L, max_seeds, group, n_qt;
  float c2;
  int64_t n_wg;  // query tiles in all
  int64_t q_sb, q_sh, q_sl, kv_sb, kv_sh, kv_sl;
};

constexpr int kFWaves = 8;  // most waves per workgroup
constexpr int kFT = 16;     // queries per workgroup, keys per tile

// WAVES: the most of a workgroup, which size its LDS
template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void cover_attn_f32_kernel(const ParamsF p) {
  constexpr int KS = D / 16, DC = D / 64;
  __shared__ __attribute__((aligned(16))) float sO[WAVES][kFT][D + 4];
  __shared__ float sM[WAVES][kFT], sL[WAVES][kFT];
  __shared__ uint32_t bits[COVER_MAX_L / 32];
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, nw = nth >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;
  const int L = p.L;
  const int n_kt = (L + kFT - 1) / kFT;

  for (int64_t li = blockIdx.x; li < p.n_wg; li += gridDim.x) {
    const int qt = (int)(li % p.n_qt);
    const int64_t bh = li / p.n_qt;
    const int h = (int)(bh % p.Hq), b = (int)(bh / p.Hq);
    const int g = h / p.group;
    const int64_t kvoff = b * p.kv_sb + g * p.kv_sh;
    const float* qbase = p.q + b * p.q_sb + h * p.q_sh;

    const int ns_raw = p.max_seeds > 0 ? p.n_seed[b] : 0;
    const int j_first = tid < p.max_seeds ? p.seed_idx[(int64_t)b * p.max_seeds + tid] : -1;
    const int qi = qt * kFT + i16;
    f32x4 qf[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
      qf[s] = *(const f32x4*)(qbase + (int64_t)min(qi, L - 1) * p.q_sl + 16 * s + 4 * g4);
    for (int w = tid; w < (L + 31) >> 5; w += nth) bits[w] = 0u;
    __syncthreads();
    const int ns = ns_raw < 0 ? 0 : (ns_raw > p.max_seeds ? p.max_seeds : ns_raw);
    if (tid < ns && (unsigned)j_first < (unsigned)L) atomicOr(&bits[j_first >> 5], 1u << (j_first & 31));
    for (int t = tid + nth; t < ns; t += nth) {
      const int j = p.seed_idx[(int64_t)b * p.max_seeds + t];
      if ((unsigned)j < (unsigned)L) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    auto is_seed = [&](int j) -> bool { return (bits[j >> 5] >> (j & 31)) & 1u; };
    const bool row_seed = qi < L && is_seed(qi);

    // one tile's operands: rows past L repeat the last (their scores are masked)
    auto load = [&](int kt, f32x4* kf, f32x4 (*vf)[DC]) __attribute__((always_inline)) {
      const int key = min(kt * kFT + i16, L - 1);
      const float* kr = (is_seed(key) ? p.kc : p.kl) + kvoff + (int64_t)key * p.kv_sl + 4 * g4;
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[s] = *(const f32x4*)(kr + 16 * s);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int kv = min(kt * kFT + 4 * g4 + r, L - 1);
        const float* vr = (is_seed(kv) ? p.vc : p.vl) + kvoff + (int64_t)kv * p.kv_sl + 4 * i16;
#pragma unroll
        for (int c = 0; c < DC; ++c) vf[r][c] = *(const f32x4*)(vr + 64 * c);
      }
    };
    // max / sum over the four lanes that share a query
    auto quad_max = [](float x) {
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      x = fmax2(__uint_as_float(a[0]), __uint_as_float(a[1]));
      return swap_max(x);
    };
    auto quad_sum = [](float x) {
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
      return swap_add(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    };
    float m = kInitMax, l = 0.0f;
    f32x4 o[DC][4];
#pragma unroll
    for (int c = 0; c < DC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[c][e] = (f32x4){};
    f32x4 kf[KS], kn[KS], vf[4][DC], vn[4][DC];
    if (wave < n_kt) load(wave, kf, vf);
    for (int kt = wave; kt < n_kt; kt += nw) {
      if (kt + nw < n_kt) load(kt + nw, kn, vn);
      f32x4 s0 = {}, s1 = {};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s][e], qf[s][e], s0, 0, 0, 0);
          s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s][e + 1], qf[s][e + 1], s1, 0, 0, 0);
        }
      float t[4], mx = kInitMax;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = kt * kFT + 4 * g4 + r;
        t[r] = (s0[r] + s1[r]) * p.c2;
        // keys past L and a seed row's own (cached) column get no weight; its live diagonal
        // term joins in the merge
        if (key >= L || (row_seed && key == qi)) t[r] = -INFINITY;
        mx = fmax2(mx, t[r]);
      }
      mx = quad_max(mx);
      const float mn = fmax2(m, mx);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int c = 0; c < DC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c][e] *= alpha;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pw = __builtin_amdgcn_exp2f(t[r] - m);
        l += pw;
#pragma unroll
        for (int c = 0; c < DC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][c][e], pw, o[c][e], 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[s] = kn[s];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < DC; ++c) vf[r][c] = vn[r][c];
    }
    // ---- merge: accumulator (c, e) register r of lane (i, g) is O[query i][64 c + 16 g + 4 r + e]
    l = quad_sum(l);
    if (g4 == 0) {
      sM[wave][i16] = m;
      sL[wave][i16] = l;
    }
#pragma unroll
    for (int c = 0; c < DC; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *(f32x4*)&sO[wave][i16][64 * c + 16 * g4 + 4 * r] = f32x4{o[c][0][r], o[c][1][r], o[c][2][r], o[c][3][r]};
    __syncthreads();
    constexpr int CH = D / 4;  // lanes per query row, 4 columns each
    for (int idx = tid; idx < kFT * CH; idx += nth) {
      const int f = idx / CH, col = 4 * (idx % CH);
      const int qr = qt * kFT + f;
      if (qr >= L) continue;  // (whole rows: the CH lanes of a row leave together)
      const bool sd = is_seed(qr);
      float mm = kInitMax, td = -INFINITY;
      f32x4 vd = {};
      for (int w = 0; w < nw; ++w) mm = fmax2(mm, sM[w][f]);
      if (sd) {
        const f32x4 qv = *(const f32x4*)(qbase + (int64_t)qr * p.q_sl + col);
        const f32x4 kd = *(const f32x4*)(p.kl + kvoff + (int64_t)qr * p.kv_sl + col);
        vd = *(const f32x4*)(p.vl + kvoff + (int64_t)qr * p.kv_sl + col);
        float dot = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(qv[e], kd[e], dot);
#pragma unroll
        for (int off = CH / 2; off >= 1; off >>= 1) dot += __shfl_xor(dot, off);
        td = dot * p.c2;
        mm = fmax2(mm, td);
      }
      const float pd = __builtin_amdgcn_exp2f(td - mm);  // 0 unless the row is a seed
      float den = pd;
      f32x4 v = vd * pd;
      for (int w = 0; w < nw; ++w) {
        const float a = __builtin_amdgcn_exp2f(sM[w][f] - mm);
        den = __builtin_fmaf(sL[w][f], a, den);
        v += *(const f32x4*)&sO[w][f][col] * a;
      }
      const float inv = 1.0f / den;
      *(f32x4*)(p.out + b * p.q_sb + h * p.q_sh + (int64_t)qr * p.q_sl + col) = v * inv;
      if (p.lse && col == 0) p.lse[bh * L + qr] = (mm + __builtin_amdgcn_logf(den)) * kLn2;
    }
    __syncthreads();  // (the next tile rebuilds the bitmap and the slots)
  }
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t stream) {
  ParamsF p;
  p.q = (const float*)a.q;
  p.kl = (const float*)a.k_live;
  p.vl = (const float*)a.v_live;
  p.kc = (const float*)a.k_cache;
  p.vc = (const float*)a.v_cache;
  p.seed_idx = a.seed_idx;
  p.n_seed = a.n_seed;
  p.out = (float*)a.out;
  p.lse = a.lse;
  p.B = a.B; p.Hq = a.Hq; p.Hkv = a.Hkv; p.L = a.L; p.max_seeds = a.max_seeds;
  p.group = a.Hq / a.Hkv;
  p.n_qt = (a.L + kFT - 1) / kFT;
  p.c2 = a.scale * 1.44269504088896341f;
  p.q_sb = a.q_sb; p.q_sh = a.q_sh; p.q_sl = a.q_sl;
  p.kv_sb = a.kv_sb; p.kv_sh = a.kv_sh; p.kv_sl = a.kv_sl;
  p.n_wg = (int64_t)a.B * a.Hq * p.n_qt;
  // Few query tiles: a wave per key tile up to 8, for the shortest chain.  From 2048 query tiles
  // the chip is full of them, and one wave that walks all keys saves the merge and LDS (43 KB at
  // d = 64: three workgroups per CU): us with 8 waves and with 1, d64: 128 heads of L 256 62 / 40,
  // 2048 of L 65 197 / 72 (192 with a lane per query row), 32 of L 256 (512 tiles) 17 / 26; d128,
  // 2048 heads of L 100 468 / 297.  Not at d = 128 past 384 keys (64 heads of L 520 174 / 203, of
  // L 250 99 / 84), where one wave's next tile arrives late.  Past 2^20 query tiles a workgroup
  // takes several.
  const int n_kt = (a.L + kFT - 1) / kFT;
  const int nw = p.n_wg >= 2048 && (a.d == 64 || n_kt <= 24) ? 1 : (n_kt < kFWaves ? n_kt : kFWaves);
  const dim3 block(64u * (unsigned)nw);
  const dim3 grid((unsigned)(p.n_wg < (1 << 20) ? p.n_wg : (1 << 20)));
  if (a.d == 128) {
    if (nw == 1) hipLaunchKernelGGL((cover_attn_f32_kernel<128, 1>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((cover_attn_f32_kernel<128, kFWaves>), grid, block, 0, stream, p);
  } else {
    if (nw == 1) hipLaunchKernelGGL((cover_attn_f32_kernel<64, 1>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((cover_attn_f32_kernel<64, kFWaves>), grid, block, 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace cover
