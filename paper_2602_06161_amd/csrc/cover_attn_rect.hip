// COVER attention for a block of queries against the whole sequence (the prefix-cache
// decoding combined with COVER in Sec. 6.6: only the current block's rows are recomputed; the
// prompt's keys and values come from the caller's cache), bf16, head size 128, on gfx950; and
// small square calls (at most 256 tiles of 32 query rows), also at head size 64.
//
// Per query row i at absolute position p = q_off + r the result is the row p of the square
// COVER attention (Sec. 5.1): keys and values of seed positions come from the cache, every
// other position's from the live tensors, and a seed row sees its own live key and value on
// its diagonal (the leave-one-out view whose closed form App. B.4 gives).
//
// With few query rows the work is bound by reading K and V, not by the MFMAs, and one
// workgroup per (row, 128-query tile) would leave most of the chip idle, so the keys are split:
//   * n_split == 1 (the default up to L = 2048): one launch, one workgroup of 8 waves per 32
//     query rows whose waves split the keys among themselves and merge in LDS (described at the
//     kernel, below).
//   * n_split > 1, two launches through the caller's workspace: the same kernel, a workgroup
//     taking one of n_split ranges of the keys and leaving per row its normalised output O / l
//     in bf16 (256 bytes) and its max and sum in fp32 (the records are written and read once, so
//     their size is traffic on top of K and V); a seed row's live diagonal term is added by the
//     split that holds the position.  Then one wave per query row merges the splits and writes O
//     and the lse.  Against a kernel of 4 waves per 128 query rows that loaded 128 keys, waited,
//     computed and loaded again (half its waves idle at 64 rows): B1 Hq32/Hkv8 L8192, 64 rows,
//     38.4 -> 21.7 us; L16000, 8 rows, 62 -> 21; B1 H12 L12000, 180 rows, 56 -> 32.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cover.h"
#include "cover_internal.h"

namespace cover {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_t;
typedef __attribute__((address_space(1))) const char gmem_t;

constexpr int kD = 128;                 // head size of the key splits' records
constexpr int kStage = 32;              // keys per stage
constexpr int kMaxWords = COVER_MAX_L / 32;
constexpr float kInit = -1.0e30f;       // finite "nothing seen yet" max
constexpr float kLn2 = 0.693147180559945309f;

struct RectParams {
  const __bf16* q;
  const __bf16* kl;
  const __bf16* vl;
  const __bf16* kc;
  const __bf16* vc;
  const int32_t* seed_idx;
  const int32_t* n_seed;
  float* ws;
  __bf16* out;
  float* lse;
  int B, Hq, Hkv, L, Lq, q_off, max_seeds, group, n_qt, n_split, split_stages;
  int n_wg, xcd_slots;  // workgroups of the launch, and of them per XCD
  float c2;  // scale * log2(e)
  int64_t q_sb, q_sh, q_sl, kv_sb, kv_sh, kv_sl;
  // key splits: first workgroup of the launch; key rows too far apart for 32-bit offsets in a stage
  int first_wg, wide;
};

// LDS layouts: K rows with the 16-byte chunk index XOR-ed by row % 16 (head size 64, two rows
// per 256-byte window: row / 2 % 8), so that a b128 operand read of 32 rows covers all banks; V
// rows with the chunk index XOR-ed by 4 (row % 4) (2 (row % 4)), so that a transposing read of 8
// rows x 64 bytes covers every bank twice.
template <int D>
__device__ __forceinline__ int k_swz(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int D>
__device__ __forceinline__ int v_swz(int row) { return (row & 3) << (D == 128 ? 2 : 1); }
template <int D>
__device__ __forceinline__ uint32_t k_off(int row, int c) { return row * (2 * D) + ((c ^ k_swz<D>(row)) << 4); }
template <int D>
__device__ __forceinline__ uint32_t v_elem(int row, int col) {
  return row * (2 * D) + (((col >> 3) ^ v_swz<D>(row)) << 4) + ((col & 7) << 1);
}

// max / sum of x over a query row's lane pair (lanes l and l ^ 32), on the VALU: the swap
// leaves one copy of each lane's own value and one of its partner's in the two results
__device__ __forceinline__ float pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ i16x4 v_tr(const lds_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)p);
}

// One wave per query row: merge the splits' (max, sum, O / sum), write O (bf16) and the lse.
__global__ __launch_bounds__(256) void cover_attn_rect_merge_kernel(const RectParams p) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // over B * Hq * Lq
  if (row >= (int64_t)p.B * p.Hq * p.Lq) return;
  const int64_t bh = row / p.Lq;
  const int r = (int)(row % p.Lq);
  const int b = (int)(bh / p.Hq), h = (int)(bh % p.Hq);
  const float* rec0 = p.ws + (bh * p.n_split * p.Lq + r) * COVER_RECT_RECORD;
  const int64_t sstride = (int64_t)p.Lq * COVER_RECT_RECORD;
  // splits in chunks of 8 whose loads are all issued before the first is used; the running
  // (max, sum, O) is rescaled between chunks
  constexpr int kChunk = 8;
  float M = kInit, den = 0.0f, o0 = 0.0f, o1 = 0.0f;
  for (int s0 = 0; s0 < p.n_split; s0 += kChunk) {
    float ms[kChunk], ls[kChunk];
    uint32_t pr[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      ms[u] = kInit;
      ls[u] = 0.0f;
      pr[u] = 0u;
      if (s0 + u < p.n_split) {
        const float* rec = rec0 + (s0 + u) * sstride;
        ms[u] = rec[kD / 2];
        ls[u] = rec[kD / 2 + 1];
        pr[u] = ((const uint32_t*)rec)[lane];  // bf16 O of dims 2 lane, 2 lane + 1
      }
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) Mn = __builtin_fmaxf(Mn, ms[u]);
    const float a = __builtin_amdgcn_exp2f(M - Mn);
    den *= a;
    o0 *= a;
    o1 *= a;
    M = Mn;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const float w = ls[u] * __builtin_amdgcn_exp2f(ms[u] - M);
      den += w;
      o0 = __builtin_fmaf(__uint_as_float(pr[u] << 16), w, o0);
      o1 = __builtin_fmaf(__uint_as_float(pr[u] & 0xffff0000u), w, o1);
    }
  }
  const float inv = 1.0f / den;
  __bf16* op = p.out + b * p.q_sb + h * p.q_sh + (int64_t)r * p.q_sl + 2 * lane;
  op[0] = (__bf16)(o0 * inv);
  op[1] = (__bf16)(o1 * inv);
  if (p.lse && lane == 0) p.lse[row] = (M + __builtin_amdgcn_logf(den)) * kLn2;
}


// ---------------------------------------------------------------------------------------
// Single-launch form (n_split == 1): one workgroup of 8 waves per (batch, query head,
// 32-query tile).  A CU's load path, not HBM, bounds a short block (about 100 GB/s per CU),
// and the merge of key splits held by different workgroups costs a second launch; so the
// key split stays inside the workgroup: wave w takes a contiguous share of the 32-key
// stages (the first four waves more than the other four, which issue their loads after
// them) and streams them through a K slot and a V slot of its own by global-to-LDS loads (no
// barrier in the loop), each slot refilled as soon as it has been read.  The eight partial
// (max, sum, O) states and a seed row's live diagonal term are merged through LDS at the end.
// Workgroups that share a KV head are placed on one XCD, so its L2 serves their re-reads.
// ---------------------------------------------------------------------------------------
constexpr int kTW = 8;             // waves per workgroup
constexpr int kTQ = 32;            // queries per workgroup
constexpr int kTSeeds = 64 * kTW;  // seed positions fetched into LDS (the rest: plain loads)
constexpr float kLazyT = 8.0f;

// s_waitcnt immediate that waits for vmcnt <= n only
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70 | 0xf00; }

// Global -> LDS loads: lane l's 16 bytes (4 for the dword form) land at LDS byte lds + 16 l
// (+ 4 l); lds is wave-uniform.  The compiler does not track them: every read of their data
// follows an explicit vmcnt wait of the issuing wave.  A wave's loads land in issue order.
__device__ __forceinline__ uint32_t lds_addr(const void* ptr) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const lds_t*)ptr);
}
__device__ __forceinline__ void dma16(uint32_t lds, gmem_t* addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(lds), "v"((uint64_t)addr) : "memory", "m0");
}
__device__ __forceinline__ void dma16s(uint32_t lds, gmem_t* base, uint32_t voff) {  // uniform base
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// the uniform-base load for the lanes of `mask` only (exec set and restored inside the
// statement; the scalar moves and the nop keep the load behind any VALU write of its operands)
__device__ __forceinline__ void dma16m(uint32_t lds, gmem_t* base, uint32_t voff, uint64_t mask) {
  uint64_t save;
  asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %1\n\ts_mov_b32 m0, %2\n\ts_nop 1\n\t"
               "global_load_lds_dwordx4 %3, %4\n\ts_mov_b64 exec, %0"
               : "=&s"(save) : "s"(mask), "s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void dma4(uint32_t lds, gmem_t* addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
               :: "s"(lds), "v"((uint64_t)addr) : "memory", "m0");
}
// the lanes that load row k, for each set bit k: 16 k .. 16 k + 15 of 4 rows (head size 128), or
// 8 k .. 8 k + 7 of 8 rows (64; the product puts bit k of a nibble at 8 k)
template <int D>
__device__ __forceinline__ uint64_t lane_rows(uint32_t n) {
  if constexpr (D == 128) {
    const uint64_t m = (uint64_t)(n & 1u) | ((uint64_t)(n & 2u) << 15) | ((uint64_t)(n & 4u) << 30) |
                       ((uint64_t)(n & 8u) << 45);
    return (m << 16) - m;
  } else {
    const uint64_t m = (uint64_t)(((n & 15u) * 0x00204081u) & 0x01010101u) |
                       ((uint64_t)(((n >> 4) * 0x00204081u) & 0x01010101u) << 32);
    return (m << 8) - m;
  }
}
__device__ __forceinline__ gmem_t* uniform_ptr(const void* ptr) {
  const uint64_t v = (uint64_t)ptr;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (gmem_t*)(((uint64_t)hi << 32) | lo);
}

// Phase timing (a separate build of the library, -DCOVER_RECT_TIMING=1, used only to measure
// where a workgroup's time goes): lane 0 of every wave of the first kTimeWG logical
// workgroups stores the shader-clock counter at fixed points.  Slots: 0 start, 1 seed list
// and Q landed, 2 seed bitmap built, 3 first stage landed, 4 + i top of the wave's stage i
// (i < 16), 20 loop done, 21 partial states in LDS (after the barrier), 22 end.
#ifndef COVER_RECT_TIMING
#define COVER_RECT_TIMING 0
#endif
#if COVER_RECT_TIMING
constexpr int kTimeWG = 1024, kTimeSlots = 32;
__device__ uint64_t g_rect_times[kTimeWG * kTW * kTimeSlots];
#define RECT_TSTAMP(slot)                                                                        \
  do {                                                                                           \
    if (li < kTimeWG && lane == 0)                                                               \
      g_rect_times[((int64_t)li * kTW + wave) * kTimeSlots + (slot)] = __builtin_readcyclecounter(); \
  } while (0)
#else
#define RECT_TSTAMP(slot) do {} while (0)
#endif

// SPLIT: key splits (records for the merge kernel); otherwise the whole of a row's keys
// (head size 128 only)
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kTW, 1) void cover_attn_tile_kernel(const RectParams p) {
  constexpr int kRow = 2 * D;              // bytes per K/V/Q row
  constexpr int kCh = D / 8;               // 16-byte chunks per row
  constexpr int kRPL = 1024 / kRow;        // rows per 1-KiB load
  constexpr int kNL = kStage / kRPL;       // loads per stage of K (or V)
  constexpr int kSB = kStage * kRow;       // bytes of one stage of K (or V)
  constexpr uint32_t kRowMask = (1u << kRPL) - 1u;
  // per wave: a K slot and a V slot (at the end: its partial O, 32 rows of D fp32);
  // the tile's Q; the seed bitmap of the sequence; the seed list, and later in its place the
  // partial maxima and sums
  __shared__ __attribute__((aligned(1024))) char sKV[kTW][2][kSB];
  __shared__ __attribute__((aligned(1024))) char sQ[kTQ * kRow];
  __shared__ uint32_t bits[kMaxWords];
  __shared__ __attribute__((aligned(16))) int32_t sSeeds[kTSeeds];
  __shared__ __attribute__((aligned(16))) int32_t sNs[4];
  static_assert(2 * kTW * kTQ <= kTSeeds, "the partial maxima and sums fit the seed list's place");
  float (*const sM)[kTQ] = (float(*)[kTQ])sSeeds;
  float (*const sL)[kTQ] = sM + kTW;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hl = lane >> 5;

  // workgroup -> (b, h, tile); consecutive logical tiles (those of one KV head) share an XCD
  const int li = (blockIdx.x & 7) * p.xcd_slots + (blockIdx.x >> 3);
  if (li >= p.n_wg) return;
  RECT_TSTAMP(0);
  int split = 0, h, b;
  const int id = SPLIT ? p.first_wg + li : li;
  const int qt = id % p.n_qt;
  int bh = id / p.n_qt;
  if constexpr (SPLIT) {  // tile fastest, then the query heads of a KV head, then its key splits
    const int hg = bh % p.group, rest = bh / p.group, kv = rest / p.n_split;
    split = rest % p.n_split;
    bh = kv * p.group + hg;
  }
  h = bh % p.Hq;
  b = bh / p.Hq;
  const int g = h / p.group;
  const int L = p.L;
  // this workgroup's 32-key stages [sb, sb + nst) (all of them without key splits)
  const int n_stages = (L + kStage - 1) / kStage;
  const int sb = SPLIT ? split * p.split_stages : 0;
  const int nst = SPLIT ? max(min(n_stages - sb, p.split_stages), 0) : n_stages;
  // this wave's stages: waves 0-3 take 10/64 of them each, waves 4-7 (the second wave of
  // each SIMD, which loses the load path's arbitration to the first) 6/64: the measured
  // split that lets the waves finish together
  const int cw0 = wave < 4 ? 10 * wave : 40 + 6 * (wave - 4);
  const int cw1 = wave < 3 ? 10 * (wave + 1) : 40 + 6 * (wave - 3);
  const int s0 = sb + nst * cw0 / 64, s1 = sb + nst * cw1 / 64;
  const int ragged = L % kStage ? n_stages - 1 : -1;
  const int nW = (L + 31) >> 5;
  for (int w = tid; w < nW; w += 64 * kTW) bits[w] = 0u;

  // load geometry: load j of a stage covers stage rows kRPL j + lane / kCh at physical chunk
  // lane % kCh, i.e. LDS byte 1024 j + 16 lane of the slot; the source chunk is the one the
  // slot's swizzle puts there (k_swz, v_swz)
  const int64_t row_bytes = p.kv_sl * 2, stage_bytes = kStage * row_bytes;
  uint32_t offK[kNL], offV[kNL];
#pragma unroll
  for (int j = 0; j < kNL; ++j) {
    const int row = kRPL * j + lane / kCh, pc = lane % kCh;
    offK[j] = (uint32_t)(row * row_bytes) + ((pc ^ k_swz<D>(row)) << 4);
    offV[j] = (uint32_t)(row * row_bytes) + ((pc ^ v_swz<D>(row)) << 4);
  }
  const int64_t kvoff = b * p.kv_sb + g * p.kv_sh;
  const char* const klc = (const char*)(p.kl + kvoff);
  const char* const kcc = (const char*)(p.kc + kvoff);
  const char* const vlc = (const char*)(p.vl + kvoff);
  const char* const vcc = (const char*)(p.vc + kvoff);
  const uint32_t slotK = lds_addr(sKV[wave][0]), slotV = lds_addr(sKV[wave][1]);
  // one stage: every row from the live tensor, or (with seeds = the stage's seed word) a seed
  // row from the cache; rows past L clamped into the sequence
  auto ld_stage = [&](uint32_t slot, const char* live, const char* cache, const uint32_t* off, int st,
                      uint32_t seeds) __attribute__((always_inline)) {
    if (st == ragged || seeds != 0u || (SPLIT && p.wide)) {
#pragma unroll
      for (int j = 0; j < kNL; ++j) {
        const int row = kRPL * j + lane / kCh;
        const int key = min(st * kStage + row, L - 1);
        const char* src = ((seeds >> row) & 1u) ? cache : live;
        dma16(slot + 1024 * j, (gmem_t*)(src + key * row_bytes + (off[j] - (uint32_t)(row * row_bytes))));
      }
    } else {
      gmem_t* base = uniform_ptr(live + st * stage_bytes);
#pragma unroll
      for (int j = 0; j < kNL; ++j) dma16s(slot + 1024 * j, base, off[j]);
    }
  };
  auto seed_word = [&](int st) __attribute__((always_inline)) -> uint32_t {
    return __builtin_amdgcn_readfirstlane(bits[st]);
  };
  // the seed rows of the first stage again (its loads went out before the seeds were known),
  // from the cache, issued after the live loads of the same slot so that they land last; a
  // load with no seed row among its four is skipped
  auto patch = [&](uint32_t slot, const char* cache, const uint32_t* off, int st)
                   __attribute__((always_inline)) {
    const uint32_t w = seed_word(st);
    if (w == 0u) return;
    if (SPLIT && p.wide) {  // (the 32-bit offsets below do not reach: every row by its own address)
      ld_stage(slot, cache == kcc ? klc : vlc, cache, off, st, w);
      return;
    }
    gmem_t* base = uniform_ptr(cache + st * stage_bytes);
#pragma unroll
    for (int j = 0; j < kNL; ++j) {
      const uint32_t rows = (w >> (kRPL * j)) & kRowMask;
      if (rows) dma16m(slot + 1024 * j, base, off[j], lane_rows<D>(rows));
    }
  };

  // ---- prologue: the seed list, Q, and this wave's first stage from the live tensors ------
  const int64_t sbase = (int64_t)b * p.max_seeds;
  if (p.max_seeds > 0) {
    if (tid == 0) dma4(lds_addr(sNs), (gmem_t*)(p.n_seed + b));
    const int e = 64 * wave + lane;
    if (e < p.max_seeds) dma4(lds_addr((const char*)sSeeds + 256 * wave), (gmem_t*)(p.seed_idx + sbase + e));
  }
  const __bf16* qbase = p.q + b * p.q_sb + h * p.q_sh;
  if (kTQ / kRPL == kTW || wave < kTQ / kRPL) {
    const int row = kRPL * wave + lane / kCh, pc = lane % kCh;
    const int qi = min(qt * kTQ + row, p.Lq - 1);
    dma16(lds_addr(sQ + 1024 * wave), (gmem_t*)((const char*)(qbase + (int64_t)qi * p.q_sl) + ((pc ^ k_swz<D>(row)) << 4)));
  }
  if (s0 < s1) {
    ld_stage(slotK, klc, kcc, offK, s0, 0u);
    ld_stage(slotV, vlc, vcc, offV, s0, 0u);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kNL));  // the seed list and Q have landed
  } else {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  }
  RECT_TSTAMP(1);
  __syncthreads();
  if (p.max_seeds > 0) {
    int ns = sNs[0];
    ns = ns < 0 ? 0 : (ns > p.max_seeds ? p.max_seeds : ns);
    if (tid < ns && tid < kTSeeds) {
      const int j = sSeeds[tid];
      if ((unsigned)j < (unsigned)L) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    for (int t = tid + kTSeeds; t < ns; t += 64 * kTW) {  // long seed lists
      const int j = p.seed_idx[sbase + t];
      if ((unsigned)j < (unsigned)L) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
  }
  __syncthreads();
  RECT_TSTAMP(2);
  auto is_seed = [&](int j) __attribute__((always_inline)) -> bool { return (bits[j >> 5] >> (j & 31)) & 1u; };
  if (s0 < s1) {
    patch(slotK, kcc, offK, s0);
    patch(slotV, vcc, offV, s0);
  }

  // Q fragments (B operand of S^T = K Q^T): query l32, d-chunk 2 ks + hl
  bf16x8 qreg[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
    qreg[ks] = *(const __attribute__((address_space(3))) bf16x8*)((const lds_t*)sQ + k_off<D>(l32, 2 * ks + hl));
  const int qrow = min(qt * kTQ + l32, p.Lq - 1);
  const int pos = p.q_off + qrow;
  const bool row_seed = is_seed(pos);

  // the live key and value rows of the seed rows this wave finishes: lane group fq = lane / 16
  // takes query kFin wave + fq, dims kE (lane % 16) .. + kE - 1, requested now and used in the merge
  constexpr int kFin = kTQ / kTW, kE = D / 16;
  typedef uint32_t raw_t __attribute__((ext_vector_type(kE / 2)));  // kE bf16 values
  typedef __bf16 out_t __attribute__((ext_vector_type(kE)));
  const int fq = lane >> 4, fj = lane & 15;
  const int qfin = qt * kTQ + kFin * wave + fq;
  const bool fin_ok = qfin < p.Lq;
  // (with key splits the diagonal term belongs to the split that holds the position)
  const int fstage = (p.q_off + qfin) / kStage;
  const bool fseed = fin_ok && (!SPLIT || (fstage >= sb && fstage < sb + nst)) && is_seed(p.q_off + qfin);
  raw_t kd = {}, vd = {};
  if (fseed) {
    const int64_t ro = kvoff + (int64_t)(p.q_off + qfin) * p.kv_sl + kE * fj;
    kd = *(const raw_t*)(p.kl + ro);
    vd = *(const raw_t*)(p.vl + ro);
  }

  // V^T operand addresses: lane (G = lane / 16, i = lane % 16) reads keys {0..3, 8..11} + 4 (G / 2)
  // of d-block db, the key order of the S^T registers
  uint32_t vaddr[D / 32];
  {
    const int G = lane >> 4, ii = lane & 15;
    const int row = 4 * (G >> 1) + (ii >> 2);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) vaddr[db] = v_elem<D>(row, db * 32 + 16 * (G & 1) + 4 * (ii & 3));
  }
  f32x16 o[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.0f;
  float m = kInit, l = 0.0f;
  const lds_t* const kb = (const lds_t*)sKV[wave][0];
  const lds_t* const vb = (const lds_t*)sKV[wave][1];

  for (int st = s0; st < s1; ++st) {
    const bool more = st + 1 < s1;
    // K(st) has landed: younger are V(st)'s kNL loads; at the first stage everything is waited
    // for (the patches of the prologue are counted nowhere)
    if (st == s0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(kNL));
    if (st == s0) RECT_TSTAMP(3);
    if (st - s0 < 16) RECT_TSTAMP(4 + st - s0);
    bf16x8 ka[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      ka[ks] = *(const __attribute__((address_space(3))) bf16x8*)(kb + k_off<D>(l32, 2 * ks + hl));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the K slot is read: refill it
    if (more) ld_stage(slotK, klc, kcc, offK, st + 1, seed_word(st + 1));
    f32x16 sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qreg[ks], sc, 0, 0, 0);
    // register r holds key k0 + 8 (r / 4) + 4 hl + r % 4 of query qrow
    const int k0 = st * kStage;
    const bool edge = k0 + kStage > L;
    const bool diag = row_seed && pos >= k0 && pos < k0 + kStage;
    float mx = kInit;
    if (__builtin_amdgcn_ballot_w64(diag) != 0 || edge) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + 8 * (r >> 2) + 4 * hl + (r & 3);
        float t = sc[r] * p.c2;
        if (key >= L || (diag && key == pos)) t = -INFINITY;
        sc[r] = t;
        mx = __builtin_fmaxf(mx, t);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[r] *= p.c2;
        mx = __builtin_fmaxf(mx, sc[r]);
      }
    }
    mx = pair_max(mx);
    if (st == s0) {
      m = mx;
    } else if (__builtin_amdgcn_ballot_w64(mx > m + kLazyT)) {
      const float mn = __builtin_fmaxf(m, mx);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db) o[db] *= alpha;
      m = mn;
    }
    bf16x8 pk[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pr = __builtin_amdgcn_exp2f(sc[8 * kk + e] - m);
        l += pr;
        pk[kk][e] = (__bf16)pr;
      }
    // V(st) has landed: younger are K(st + 1)'s kNL loads, if there is a stage st + 1
    if (more) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kNL));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    bf16x8 va[2][D / 32];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        const lds_t* base = vb + vaddr[db] + kk * 16 * kRow;
        va[kk][db] = __builtin_bit_cast(
            bf16x8, __builtin_shufflevector(v_tr(base), v_tr(base + 8 * kRow), 0, 1, 2, 3, 4, 5, 6, 7));
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the V slot is read: refill it
    if (more) {
      ld_stage(slotV, vlc, vcc, offV, st + 1, seed_word(st + 1));
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[kk][db], pk[kk], o[db], 0, 0, 0);
  }

  // ---- merge: every wave's (max, sum, O) through LDS ---------------------------------------
  // O goes to this wave's own slots (its loads have all landed and been read): row l32, 16-byte
  // chunk c (dims 4 c .. 4 c + 3) at byte 4 D l32 + 16 (c ^ l32 % (D / 4))
  RECT_TSTAMP(20);
  constexpr int kOM = D / 4 - 1;
  const float lt = pair_sum(l);
  if (hl == 0) {
    sM[wave][l32] = m;
    sL[wave][l32] = lt;
  }
  {
    lds_t* const ob = (lds_t*)sKV[wave][0] + 4 * D * l32;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c = 8 * db + 2 * gq + hl;
        *(__attribute__((address_space(3))) f32x4*)(ob + ((c ^ (l32 & kOM)) << 4)) =
            f32x4{o[db][4 * gq], o[db][4 * gq + 1], o[db][4 * gq + 2], o[db][4 * gq + 3]};
      }
  }
  __syncthreads();
  RECT_TSTAMP(21);
  // wave w finishes queries kFin w + fq (lane group fq), lane dims kE fj .. kE fj + kE - 1; every
  // LDS read of the merge is requested before the first is used
  {
    const int f = kFin * wave + fq;
    float mw[kTW], lw[kTW];
    f32x4 ow[kTW][kE / 4];
#pragma unroll
    for (int w = 0; w < kTW; ++w) {
      mw[w] = sM[w][f];
      lw[w] = sL[w][f];
      const lds_t* rb = (const lds_t*)sKV[w][0] + 4 * D * f;
#pragma unroll
      for (int u = 0; u < kE / 4; ++u)
        ow[w][u] = *(const __attribute__((address_space(3))) f32x4*)(rb + (((kE / 4 * fj + u) ^ (f & kOM)) << 4));
    }
    const raw_t qv = *(const __attribute__((address_space(3))) raw_t*)(
        (const lds_t*)sQ + k_off<D>(f, kE * fj / 8) + 2 * (kE * fj % 8));
    float M = kInit;
#pragma unroll
    for (int w = 0; w < kTW; ++w) M = __builtin_fmaxf(M, mw[w]);
    // the live diagonal score q . k_live(pos) of a seed row (App. B.4), summed over the
    // group's 16 lanes
    float dot = 0.0f;
#pragma unroll
    for (int e = 0; e < kE / 2; ++e) {
      dot = __builtin_fmaf(__uint_as_float(qv[e] << 16), __uint_as_float(kd[e] << 16), dot);
      dot = __builtin_fmaf(__uint_as_float(qv[e] & 0xffff0000u), __uint_as_float(kd[e] & 0xffff0000u), dot);
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) dot += __shfl_xor(dot, off);
    const float t = dot * p.c2;
    if (fseed) M = __builtin_fmaxf(M, t);
    float den = 0.0f, acc[kE];
#pragma unroll
    for (int e = 0; e < kE; ++e) acc[e] = 0.0f;
#pragma unroll
    for (int w = 0; w < kTW; ++w) {
      const float a = __builtin_amdgcn_exp2f(mw[w] - M);
      den = __builtin_fmaf(lw[w], a, den);
#pragma unroll
      for (int e = 0; e < kE; ++e) acc[e] = __builtin_fmaf(a, ow[w][e >> 2][e & 3], acc[e]);
    }
    if (fseed) {
      const float pd = __builtin_amdgcn_exp2f(t - M);
      den += pd;
#pragma unroll
      for (int e = 0; e < kE / 2; ++e) {
        acc[2 * e] = __builtin_fmaf(pd, __uint_as_float(vd[e] << 16), acc[2 * e]);
        acc[2 * e + 1] = __builtin_fmaf(pd, __uint_as_float(vd[e] & 0xffff0000u), acc[2 * e + 1]);
      }
    }
    if (SPLIT && fin_ok) {  // the split's record: O / sum in bf16, the max and the sum
      float* rec = p.ws + (((int64_t)bh * p.n_split + split) * p.Lq + qfin) * COVER_RECT_RECORD;
      const float inv = den > 0.0f ? 1.0f / den : 0.0f;
      out_t ob;
#pragma unroll
      for (int e = 0; e < kE; ++e) ob[e] = (__bf16)(acc[e] * inv);
      *(out_t*)((__bf16*)rec + kE * fj) = ob;
      if (fj == 0) {
        rec[D / 2] = M;
        rec[D / 2 + 1] = den;
      }
    } else if (fin_ok) {
      const float inv = 1.0f / den;
      out_t ob;
#pragma unroll
      for (int e = 0; e < kE; ++e) ob[e] = (__bf16)(acc[e] * inv);
      *(out_t*)(p.out + b * p.q_sb + h * p.q_sh + (int64_t)qfin * p.q_sl + kE * fj) = ob;
      if (p.lse && fj == 0) p.lse[(int64_t)bh * p.Lq + qfin] = (M + __builtin_amdgcn_logf(den)) * kLn2;
    }
  }
  RECT_TSTAMP(22);
}

}  // namespace

#if COVER_RECT_TIMING
// Copies the timing slots of the last launch of the single-launch kernel (layout
// [workgroup][wave][slot], 1024 x 8 x 32 values) to host memory; waits for the device.  Only
// in the timing build of the library.
extern "C" int cover_rect_timing_read(uint64_t* host, int64_t n) {
  const int64_t cap = (int64_t)kTimeWG * kTW * kTimeSlots;
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(g_rect_times), sizeof(uint64_t) * (n < cap ? n : cap),
                                  0, hipMemcpyDeviceToHost);
}
#endif

// One round of workgroups of 32 query rows is always shorter than the four-wave kernel's round
// of 128 (us, d128 Hq32: L100 6.9 against 10.9, L256 7.1 against 12.9; Hq12 L600 9.3 against
// 18.5; d64 Hq32: L100 5.4 against 8.1, L256 6.1 against 9.9; Hq12 L600 6.8 against 13.5), two
// rounds are not (Hq32 L512 d128 17.0 against 16.4, d64 12.0 against 11.9; four rounds at L1024
// d128 40 against 24), because every 32 rows read all the keys again.  (At 64 two workgroups
// per CU would fit the LDS, but not the registers: spilling, one round takes 7.5-9.)
bool attn_small(const AttnArgs& a) {
  return (int64_t)a.B * a.Hq * ((a.L + kTQ - 1) / kTQ) <= 256 &&
         a.kv_sl < (int64_t(1) << 26);
}

// The key ranges a call with n_split of them uses: all, unless fewer finish sooner.  A tile of 32
// query rows reads its range of the keys for itself, so splitting past the point where the
// workgroups fill the chip only adds rounds and records.  Cost in 32-key stages, as measured: rounds
// of 256 workgroups, each as long as its stages and 18 more for its start and merge; 24 for the
// second launch.  Asked for 64 ranges at B1 Hq32 L8192, 64 rows: 100 us with all of them, 57 on the
// former kernel of 4 waves per 128 rows, 21.8 with the 4 that this picks; 4 ranges at B1 Hq32 L1024, 256
// rows: 34, 23.3, 12.1 with one.
static int rect_ranges(int64_t tiles, int stages, int n_split, bool whole) {
  int best = n_split;
  int64_t least = INT64_MAX;
  auto offer = [&](int64_t n) {
    if (n < (whole ? 1 : 2) || n > n_split) return;
    const int length = (int)((stages + n - 1) / n);
    const int64_t cost = (tiles * n + 255) / 256 * (length + 18) + (n > 1 ? 24 : 0);
    if (cost < least) {
      best = (int)n;
      least = cost;
    }
  };
  offer(n_split);
  for (int rounds = 1; rounds <= 8; ++rounds) offer(256 * rounds / tiles);
  offer(2);
  offer(1);
  return best;
}

hipError_t launch_attn_rect(const RectArgs& a, hipStream_t stream) {
  RectParams p;
  p.q = (const __bf16*)a.q; p.kl = (const __bf16*)a.k_live; p.vl = (const __bf16*)a.v_live;
  p.kc = (const __bf16*)a.k_cache; p.vc = (const __bf16*)a.v_cache;
  p.seed_idx = a.seed_idx; p.n_seed = a.n_seed; p.ws = a.workspace;
  p.out = (__bf16*)a.out; p.lse = a.lse;
  p.B = a.B; p.Hq = a.Hq; p.Hkv = a.Hkv; p.L = a.L; p.Lq = a.Lq; p.q_off = a.q_off;
  p.max_seeds = a.max_seeds; p.group = a.Hq / a.Hkv;
  p.n_qt = (a.Lq + kTQ - 1) / kTQ;
  const int stages = (a.L + kStage - 1) / kStage;
  const int64_t tiles = (int64_t)a.B * a.Hq * p.n_qt;
  constexpr int64_t kMaxGrid = (int64_t(1) << 23) - 8;  // workgroups per launch: under 2^32 work-items
  p.wide = a.kv_sl >= (int64_t(1) << 26);
  p.n_split = rect_ranges(tiles, stages, a.n_split, !p.wide && tiles <= kMaxGrid);
  p.split_stages = (stages + p.n_split - 1) / p.n_split;
  p.c2 = a.scale * 1.44269504088896341f;
  p.q_sb = a.q_sb; p.q_sh = a.q_sh; p.q_sl = a.q_sl;
  p.kv_sb = a.kv_sb; p.kv_sh = a.kv_sh; p.kv_sl = a.kv_sl;
  const int64_t n = tiles * p.n_split;
  const dim3 block(64 * kTW);
  if (p.n_split == 1) {
    p.n_wg = (int)n;
    p.xcd_slots = (int)((n + 7) / 8);
    const dim3 grid((unsigned)(8 * (int64_t)p.xcd_slots));
    if (a.d == 128) hipLaunchKernelGGL((cover_attn_tile_kernel<128, false>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((cover_attn_tile_kernel<64, false>), grid, block, 0, stream, p);
    return hipGetLastError();
  }
  for (int64_t first = 0; first < n; first += kMaxGrid) {
    p.first_wg = (int)first;
    p.n_wg = (int)(n - first < kMaxGrid ? n - first : kMaxGrid);
    p.xcd_slots = (p.n_wg + 7) / 8;
    hipLaunchKernelGGL((cover_attn_tile_kernel<128, true>), dim3((unsigned)(8 * p.xcd_slots)), block, 0, stream, p);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t rows = (int64_t)a.B * a.Hq * a.Lq;
  hipLaunchKernelGGL(cover_attn_rect_merge_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace cover
