// Temperature sampling of the draft tokens on gfx950 (the stochastic decoding the paper tests
// in its appendix on robustness, T in {0.1, 0.2, 0.3}).
//
// Per row of logits x (one workgroup per row, one pass over the row):
//   token = argmax_v (x_v / T + g_v),  g_v = -ln(-ln u_v)   (Gumbel-max: token ~ softmax(x/T))
//   p     = softmax(x / T) at the token (the confidence the drafting threshold compares)
// u_v is word v % 4 of Philox4x32-10 (Salmon et al., SC 2011) at counter (v / 4, row, step, 0)
// and key (seed mod 2^32, seed / 2^32), mapped to ((w >> 9) + 1/2) 2^-23, so every (row,
// token, step) has its own fixed random number whatever the launch shape.  The argmax is
// taken as the equivalent exponential race (below).
//
// What bounds it: the generator.  Ten Philox rounds, a logarithm and an exponential for every
// token of 256 rows of 126464 is 38 us of vector ALU work, against 13 us for reading the bf16
// logits.  But a token can only be drawn if its z = x / T comes within the largest Gumbel value
// (16.3 in natural units: u has 23 bits) of the best perturbed score so far, so the generator
// runs only for the quads of tokens (one Philox call) that reach that bound: each wave queues
// them in LDS and races 64 at a time, so that no lane idles.  The bound starts at the row's
// largest early logit less the smallest Gumbel value and rises as better tokens are found.
// For flat rows nearly every quad qualifies; then they are raced where they are (the queue
// would only cost).  The race itself needs neither a logarithm nor an exponential for the
// tokens that cannot beat the best score so far, which is nearly all.  Measured, 256 rows of
// 126464 bf16 logits N(0, 2^2) with a raised token, against running the generator for every
// token: T = 0.1 38.3 -> 18.0 us, T = 0.3 38.1 -> 22.4, T = 1 38.1 -> 31.4.  In the last round of
// loads only what a wave has is worked on (2048 rows of 1000: 21.5 us, 28.5 when the padding
// was folded and offered like the rest, 18.8 now).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cover.h"
#include "cover_internal.h"

namespace cover {
namespace {

template <int N>
struct IC {
  static constexpr int value = N;
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 gu32x4;

struct SampleParams {
  const char* logits;
  int32_t* token;
  float* prob;
  int64_t row_stride_bytes;
  int V;
  float c;  // log2 e / T
  double c64;
  uint32_t k0, k1, step;
};

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
// Philox4x32-10: ten rounds; each multiplies counter words 0 and 2 by the two round
// constants and mixes the 64-bit products' halves with words 1 and 3 and the key, which is
// advanced by the Weyl constants between rounds.
__device__ __forceinline__ u32x4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                        uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    const uint32_t n0 = xor3(hi1, c1, k0), n2 = xor3(hi0, c3, k1);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  return u32x4{c0, c1, c2, c3};
}

// The Gumbel-max draw argmax_v (z_v - ln(-ln u_v)), z = x / T, as an exponential race: with
// E_v = -log2 u_v (1 / ln 2 times an Exp(1) variable) the token with the largest score
// z_v / ln 2 - log2 E_v wins, the smaller index on equal scores.  The score is a number of the
// token alone, so who wins does not depend on who meets whom in which order, and it is formed in
// 64 bits (the logarithm from E's exponent and, in fp32, its mantissa), which the few tokens that
// come this far afford: to 2^-22 whatever the size of z.
__device__ __forceinline__ float race_e(uint32_t w) {  // -log2 u > 0
  const float u = __builtin_fmaf((float)(w >> 9), 1.1920928955078125e-7f, 5.9604644775390625e-8f);  // ((w >> 9) + 1/2) 2^-23
  return -__builtin_amdgcn_logf(u);
}
__device__ __forceinline__ double score(float x, float E, double c64) {
  const double l = (double)__builtin_amdgcn_frexp_expf(E) + (double)__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(E));
  return __builtin_fma((double)x, c64, -l);
}
// scores are z / ln 2 - log2 E: the largest and smallest -log2 E (u = 1 - 2^-24 and 2^-24)
constexpr float kMaxAdvantage = 23.48f;
constexpr float kMinAdvantage = -4.585f;

struct Acc {
  double sc;  // the best token so far: its score
  float bx;   // its logit
  int i;      // its index
  float nm;   // reference of the sum: -m c rounded once, m the largest logit (at least kFloor)
  float s;    // sum of exp2(x c + nm)
};
__device__ __forceinline__ bool beats(double sc, int i, const Acc& a) { return sc > a.sc || (sc == a.sc && i < a.i); }

// the reference of the sum never goes below this, so that a first chunk of masked logits (-inf,
// or the type's lowest value) adds zeros and not NaN
constexpr float kFloor = -1.0e30f;

// The factor that takes a sum from reference nm to nn <= nm: the difference of the two rounded
// references, so that every term of the row's sum has the same one and its rounding cancels in the
// quotient at the end (a row's largest term is then exactly the numerator of its token: no
// probability above 1).  Both infinite, from products beyond fp32: the sum is 0 and stays it.
__device__ __forceinline__ float rescale(float nm, float nn) {
#pragma clang fp contract(off)
  return __builtin_amdgcn_exp2f(fminf(nn - nm, 0.0f));
}
__device__ __forceinline__ Acc merge(Acc a, Acc b) {
  const float nm = fminf(a.nm, b.nm);
  a.s = a.s * rescale(a.nm, nm) + b.s * rescale(b.nm, nm);
  a.nm = nm;
  if (beats(b.sc, b.i, a)) {
    a.sc = b.sc;
    a.bx = b.bx;
    a.i = b.i;
  }
  return a;
}

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// fp32 <-> int with the same order (no NaN)
__device__ __forceinline__ int order_int(float f) {
  const int i = __float_as_int(f);
  return i ^ ((i >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float order_float(int i) { return __int_as_float(i ^ ((i >> 31) & 0x7fffffff)); }

// the wave's largest value, in every lane (x is never NaN)
__device__ __forceinline__ float wave_max(float x) {
  auto step = [&](auto ctrl) __attribute__((always_inline)) {
    const int v = __float_as_int(x);
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(v, v, decltype(ctrl)::value, 0xf, 0xf, false)));
  };
  step(IC<0x111>{});  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has the row's
  step(IC<0x112>{});
  step(IC<0x114>{});
  step(IC<0x118>{});
  step(IC<0x142>{});  // row_bcast 15 and 31: lane 63 has the wave's
  step(IC<0x143>{});
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

constexpr int kDense = 48;       // lanes from which a quad is raced in place instead of queued
constexpr int kQueue = 63 + kDense - 1;  // a wave's queue: up to 63 left over, kDense - 1 pushed

// kThreads threads per row, kUnroll 16-byte loads per thread in flight
template <bool BF, int kThreads, int kUnroll>
__global__ __launch_bounds__(kThreads, 4) void cover_token_sample_kernel(const SampleParams p) {
#pragma clang fp contract(off)  // (the sum's references are rounded once, where they are formed)
  constexpr int N = BF ? 8 : 4;   // elements per 16-byte chunk
  constexpr int QPC = N / 4;      // quads per chunk
  constexpr int W = BF ? 2 : 4;   // 32-bit words per quad
  __shared__ Acc red[kThreads / 64];
  __shared__ uint32_t q_id[kThreads / 64][kQueue];
  __shared__ uint32_t q_raw[kThreads / 64][W][kQueue];
  __shared__ int s_best;  // the best perturbed score of the row so far (log2 units, order_int)
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const char* row = p.logits + (int64_t)r * p.row_stride_bytes;
  const int nfull = p.V / N;
  const float c = p.c;  // x -> log2 units
  const float rc = 1.0f / c;
  if (tid == 0) s_best = order_int(-INFINITY);
  __syncthreads();

  float m = kFloor;  // the largest logit of this thread (at least kFloor)
  Acc acc = {-INFINITY, -INFINITY, 0x7fffffff, -(kFloor * c), 0.0f};
  float best = -INFINITY, xmin = -INFINITY;  // the row's best score known here; logits below xmin cannot win
  auto values = [&](const uint32_t* w, float* x) __attribute__((always_inline)) {
    if constexpr (BF) {
      x[0] = bf_lo(w[0]); x[1] = bf_hi(w[0]); x[2] = bf_lo(w[1]); x[3] = bf_hi(w[1]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(w[e]);
    }
  };
  auto race1 = [&](float x, float E, int v) __attribute__((always_inline)) {
    const double sc = score(x, E, p.c64);
    if (beats(sc, v, acc)) {
      acc.sc = sc;
      acc.bx = x;
      acc.i = v;
    }
  };
  // The bounds that follow from `best`, slackened by the rounding of the scores (2^-24 of their
  // size in each operation): xmin, and the offset of the test in `race`.
  // Where the products leave fp32's range (c or the scores beyond kWild) nothing is skipped by
  // the second, and the first counts from the largest finite score.
  constexpr float kWild = 1.0e30f, kMaxFloat = 3.402823466e38f;
  const bool wild = !(c < kWild);
  const float c23 = wild ? 0.0f : c * 8388608.0f;
  float k23 = INFINITY;
  auto set_bound = [&]() __attribute__((always_inline)) {
    best = fminf(best, kMaxFloat);
    const float slack = 0.0625f + 1.0e-5f * __builtin_fabsf(best);
    xmin = (best - kMaxAdvantage - slack) * rc;
    k23 = wild || !(__builtin_fabsf(best) < kWild) ? INFINITY : (127.0f - best + slack) * 8388608.0f;
  };
  // The race of this lane's quad (lanes with `on`).  A token takes part only if its score
  // reaches the row's best, E <= 2^t with t = z / ln 2 - best.  Without a logarithm or an
  // exponential: 2^t <= U, the float whose bits are (t + 127) 2^23 (1 + f >= 2^f), and
  // E ln 2 = -ln u >= 1 - u, so a token with 1 - u > U ln 2 is out (its u compared as w 2^-32,
  // which is within 2^-23 of it).  What remains, a few tokens per row, is raced exactly.
  auto race = [&](uint32_t q, const uint32_t* w, bool on) __attribute__((always_inline)) {
    const u32x4 rnd = philox(q, r, p.step, 0u, p.k0, p.k1);
    float x[4];
    values(w, x);
    constexpr float kTwo32 = 4294967296.0f, kLn2Up = 0.69322f;
    constexpr float kIn = (1.0f - 3.0e-7f) * kTwo32;
    float y[4], top = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // (at most 2^127; a NaN, from a row without a bound yet, takes part; a conversion of less
      // than 0 is undefined)
      const float t = fmaxf(fminf(__builtin_fmaf(x[e], c23, k23), 2130706432.0f), 0.0f);
      y[e] = __builtin_fmaf(__uint_as_float((uint32_t)t), kLn2Up * kTwo32, (float)rnd[e]);
      top = fmaxf(top, y[e]);
    }
    const bool in = on && top >= kIn;
    if (__builtin_amdgcn_ballot_w64(in) == 0) return;
    if (in) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (y[e] >= kIn) race1(x[e], race_e(rnd[e]), 4 * (int)q + e);
    }
    const float sc = (float)acc.sc;
    if (__builtin_amdgcn_ballot_w64(sc > best) == 0) return;
    best = wave_max(sc);
    if (lane == 0) atomicMax(&s_best, order_int(best));
    set_bound();
  };
  auto see_best = [&]() __attribute__((always_inline)) {
    const float seen = order_float(*(volatile int*)&s_best);
    if (seen > best) {
      best = seen;
      set_bound();
    }
  };
  int qn = 0;  // entries of this wave's queue
  auto offer = [&](uint32_t q, const uint32_t* w, float mx) __attribute__((always_inline)) {
    const bool f = mx >= xmin;
    const uint64_t mask = __builtin_amdgcn_ballot_w64(f);
    const int n = __builtin_popcountll(mask);
    if (n == 0) return;
    uint32_t rq = q, rw[W];
#pragma unroll
    for (int k = 0; k < W; ++k) rw[k] = w[k];
    bool on = f;
    if (n < kDense) {
      const int at = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (f) {
        q_id[wave][at] = q;
#pragma unroll
        for (int k = 0; k < W; ++k) q_raw[wave][k][at] = w[k];
      }
      qn += n;
      if (qn < 64) return;
      qn -= 64;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      rq = q_id[wave][qn + lane];
#pragma unroll
      for (int k = 0; k < W; ++k) rw[k] = q_raw[wave][k][qn + lane];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      on = true;
    }
    race(rq, rw, on);
  };
  // the sum of exponentials over one chunk; returns the largest logit of each quad
  auto fold = [&](const u32x4& raw, float* mx) __attribute__((always_inline)) {
#pragma clang fp contract(off)
    float x[N];
    float cm = kFloor;
#pragma unroll
    for (int k = 0; k < QPC; ++k) {
      const uint32_t w[4] = {raw[(k * W) & 3], raw[(k * W + 1) & 3], raw[2], raw[3]};
      values(w, x + 4 * k);
      mx[k] = fmaxf(fmaxf(fmaxf(x[4 * k], x[4 * k + 1]), x[4 * k + 2]), x[4 * k + 3]);
      cm = fmaxf(cm, mx[k]);
    }
    m = fmaxf(m, cm);
    const float nm = -(m * c);
    float t[N / 2];
#pragma unroll
    for (int e = 0; e < N / 2; ++e)
      t[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * e], c, nm)) +
             __builtin_amdgcn_exp2f(__builtin_fmaf(x[2 * e + 1], c, nm));
    float sum = t[0];
#pragma unroll
    for (int e = 1; e < N / 2; ++e) sum += t[e];
    acc.s = acc.s * rescale(acc.nm, nm) + sum;
    acc.nm = nm;
  };
  // (unconditional loads, so that a round's loads stay in flight across the work on the round
  // before; a chunk past the end repeats the last one and is blanked to -inf below)
  auto load = [&](int c0, u32x4* v) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      v[u] = *(gu32x4*)((__attribute__((address_space(1))) const char*)row + (int64_t)min(c0 + u * kThreads, nfull - 1) * 16);
  };

  constexpr int kRound = kThreads * kUnroll;
  constexpr uint32_t kBlank = BF ? 0xff80ff80u : 0xff800000u;
  u32x4 cur[kUnroll], nxt[kUnroll];
  if (nfull > 0) load(tid, cur);
  for (int c0 = tid; c0 - tid < nfull; c0 += kRound) {
    load(c0 + kRound, nxt);
    if (c0 - tid + kRound > nfull) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        if (c0 + u * kThreads >= nfull) cur[u] = (u32x4){kBlank, kBlank, kBlank, kBlank};
    }
    const int first = __builtin_amdgcn_readfirstlane(c0 - lane);  // (uniform: this wave's first chunk)
    float mx[kUnroll][QPC];
    if (c0 - tid + kRound <= nfull) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) fold(cur[u], mx[u]);
    } else {  // the last round: chunks that no lane of the wave has cost nothing
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if (first + u * kThreads < nfull) {
          fold(cur[u], mx[u]);
        } else {
#pragma unroll
          for (int k = 0; k < QPC; ++k) mx[u][k] = -INFINITY;
        }
      }
    }
    if (c0 == tid) {  // the first bound of the row: its largest logit so far, with the least u
      float top = -INFINITY;
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
#pragma unroll
        for (int k = 0; k < QPC; ++k)
          top = fmaxf(top, mx[u][k]);
      top = wave_max(top);
      if (lane == 0) atomicMax(&s_best, order_int(top > kFloor ? top * c + kMinAdvantage : -INFINITY));
      __syncthreads();
    }
    see_best();
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (first + u * kThreads >= nfull) break;
#pragma unroll
      for (int k = 0; k < QPC; ++k) {
        uint32_t w[W];
#pragma unroll
        for (int e = 0; e < W; ++e) w[e] = cur[u][k * W + e];
        offer((uint32_t)(c0 + u * kThreads) * QPC + k, w, mx[u][k]);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) cur[u] = nxt[u];
  }
  __syncthreads();
  see_best();
  if (qn > 0) {  // what is left in the queue and can still win
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t v[W] = {};
    uint32_t q = 0;
    bool on = false;
    if (lane < qn) {
      q = q_id[wave][lane];
#pragma unroll
      for (int k = 0; k < W; ++k) v[k] = q_raw[wave][k][lane];
      float x[4];
      values(v, x);
      on = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])) >= xmin;
    }
    if (__builtin_amdgcn_ballot_w64(on) != 0) race(q, v, on);
  }
  auto element = [&](int v) __attribute__((always_inline)) -> float {
    return BF ? __uint_as_float((uint32_t)((const uint16_t*)row)[v] << 16) : ((const float*)row)[v];
  };
  // the tail: one element per thread, read at its own width
  if (tid < p.V - nfull * N) {
    const int v = nfull * N + tid;
    const float x = element(v);
    const u32x4 w = philox((uint32_t)(v >> 2), r, p.step, 0u, p.k0, p.k1);
    const float nm = -(fmaxf(m, x) * c);
    acc.s = acc.s * rescale(acc.nm, nm) + __builtin_amdgcn_exp2f(__builtin_fmaf(x, c, nm));
    acc.nm = nm;
    race1(x, race_e(w[v & 3]), v);
  }
  // merge: across the wave, then the waves
  auto wave_merge = [&](Acc a) __attribute__((always_inline)) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      Acc b;
      b.bx = __shfl_xor(a.bx, o);
      b.sc = __shfl_xor(a.sc, o);
      b.i = __shfl_xor(a.i, o);
      b.nm = __shfl_xor(a.nm, o);
      b.s = __shfl_xor(a.s, o);
      a = merge(a, b);
    }
    return a;
  };
  acc = wave_merge(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (wave == 0) {
    Acc a = lane < kThreads / 64 ? red[lane] : Acc{-INFINITY, -INFINITY, 0x7fffffff, -(kFloor * c), 0.0f};
    a = wave_merge(a);
    float top = __builtin_amdgcn_exp2f(__builtin_fmaf(a.bx, c, a.nm));
    if (a.s == 0.0f && p.prob) {
      // every logit of the row is below kFloor: the sum again, relative to the token drawn
      float s = 0.0f;
      for (int v = lane; v < p.V; v += 64) s += __builtin_amdgcn_exp2f((element(v) - a.bx) * c);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
      a.s = s;
      top = 1.0f;
    }
    if (lane == 0) {
      p.token[r] = a.i < p.V ? a.i : 0;  // (no token, no race: only NaN in the row)
      if (p.prob) p.prob[r] = top / a.s;
    }
  }
}

}  // namespace

hipError_t launch_token_sample(const SampleArgs& a, hipStream_t stream) {
  SampleParams p;
  p.logits = (const char*)a.logits;
  p.token = a.token;
  p.prob = a.prob;
  p.row_stride_bytes = a.row_stride * (a.bf16 ? 2 : 4);
  p.V = a.V;
  p.c64 = 1.4426950408889634 / (double)a.temperature;
  p.c = p.c64 < 0x1p127 ? (float)p.c64 : 0x1p127f;  // (infinite below T = 2^-128: then 0 c was NaN)
  p.k0 = (uint32_t)(a.seed & 0xffffffffu);
  p.k1 = (uint32_t)(a.seed >> 32);
  p.step = a.step;
  // Up to one row per CU: 1024 threads.  More rows: 512 threads of the same registers each, so
  // that two rows share a CU (1024 at these registers fill one).  256 rows of 126464, T = 0.3:
  // 22.4 us with 1024 threads, 24.8 with 512; 512 rows: 40.7 against 36.2; 300 rows of 32000 at
  // T = 0.2 / 1.0: 15.5 / 23.8 against 12.6 / 19.7.
  const dim3 grid((unsigned)a.R);
  if (a.R <= 256) {
    if (a.bf16) hipLaunchKernelGGL((cover_token_sample_kernel<true, 1024, 2>), grid, dim3(1024), 0, stream, p);
    else hipLaunchKernelGGL((cover_token_sample_kernel<false, 1024, 2>), grid, dim3(1024), 0, stream, p);
  } else {
    if (a.bf16) hipLaunchKernelGGL((cover_token_sample_kernel<true, 512, 4>), grid, dim3(512), 0, stream, p);
    else hipLaunchKernelGGL((cover_token_sample_kernel<false, 512, 4>), grid, dim3(512), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace cover
