// Compressor of one APB host (Sec. 3.4; Alg. 2, compression step) for gfx950:
// ArgTop-l_p of the retaining-head scores of every KV head, then the gather
// K^C = K_h[idx], V^C = V_h[idx].
//
// Design.  S workgroups per KV head; every one of them first finds the head's
// selection threshold (the l_p-th largest score, as an order-preserving
// 32-bit key) and the number selected before each range of indices, then
// lists and gathers the rows of its own share of the output positions, in
// index order (ascending output, lower index wins ties), with 16-byte copies.
// Each repeats the same selection over the head's scores, which stay in L2,
// so no scratch memory, atomics across workgroups or second launch are
// needed.  Local blocks up to kRegMaxKeys hold their keys in registers, longer
// ones stream them.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "apb_internal.h"

namespace apb {
namespace {

// Order-preserving map of an fp32 score to an unsigned key: a larger score
// gives a larger key, -0 maps with +0, NaN maps to 0 (below -inf, whose key
// is 0x007fffff).
__device__ __forceinline__ uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The score of a key that some score has (of -0 and +0: +0); of other keys, a
// NaN above +inf.
__device__ __forceinline__ float key_score(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
}

// ---------------------------------------------------------------------------
// Register-resident form, for Lb <= 1024 * KPT.  1024 threads; thread t holds
// the keys of local indices KPT*t .. KPT*t + KPT-1, loaded once with 16-byte
// vector loads.  The radix select takes three digits of 11, 11 and 10 bits,
// each counted into one shared 2048-bin histogram (wider digits spread the
// keys of one wave's atomics over more addresses and save a pass); the
// selected counts before each thread's range come from a block scan.
// Workgroup c of a head then gathers the selected rows whose output positions
// fall in its share [c*lp/S, (c+1)*lp/S).
constexpr int kRegThreads = 1024;
constexpr int kRegWaves = kRegThreads / 64;
constexpr int kSelBins = 2 * kRegThreads;  // 11-bit digits, two bins per thread
// Longest block of the register kernel: with 16 keys per thread it takes 13.8 us
// where the streaming one takes 17.5 (16384 N(0,1) scores, 8 KV heads, l_p =
// Lb / 8); with 32 keys per thread (and 64, half of them in LDS) it took 22.7
// against 19.6 us at 20000, 27.6 against 23.5 at 32768, 54.6 against 37.3 at
// 65536.
constexpr int kRegMaxKeys = 16 * kRegThreads;

// Inclusive prefix sum over the 64 lanes of a wave: shifts inside each
// 16-lane row through DPP, then the three row totals taken by readlane.
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
  const int row = (threadIdx.x & 63) >> 4;
  return x + (row >= 1 ? r0 : 0u) + (row >= 2 ? r1 : 0u) + (row >= 3 ? r2 : 0u);
}

template <int KPT>
__global__ void __launch_bounds__(kRegThreads)
topk_gather_reg_kernel(const float* __restrict__ scores, const uint16_t* __restrict__ k,
                       const uint16_t* __restrict__ v, int32_t* __restrict__ out_idx,
                       uint16_t* __restrict__ out_k, uint16_t* __restrict__ out_v, int La,
                       int Lb, int lp, int head_dim, int share) {
  __shared__ uint32_t hist[kSelBins];
  __shared__ uint32_t wtot[kRegWaves];
  __shared__ uint32_t wsum_gt[kRegWaves], wsum_eq[kRegWaves];
  __shared__ uint32_t sel_digit, sel_above;
  __shared__ int32_t list_src[1024];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int head = blockIdx.y;
  const float* s = scores + (size_t)head * Lb;
  const int i0 = KPT * tid;

  // ---- keys in registers; indices past Lb are marked invalid
  uint32_t key[KPT];
  if (i0 + KPT <= Lb && ((uintptr_t)s & 15u) == 0) {
#pragma unroll
    for (int j = 0; j < KPT; j += 4) {
      const float4 f = *reinterpret_cast<const float4*>(s + i0 + j);
      key[j] = score_key(f.x); key[j + 1] = score_key(f.y);
      key[j + 2] = score_key(f.z); key[j + 3] = score_key(f.w);
    }
  } else {
#pragma unroll
    for (int j = 0; j < KPT; ++j) key[j] = i0 + j < Lb ? score_key(s[i0 + j]) : 0u;
  }
  const int n_valid = max(0, min(KPT, Lb - i0));

  // every share slot is filled below (exactly lp distinct positions are
  // selected); -1 marks a slot as empty for the gather regardless
  list_src[tid] = -1;

  // ---- 1. radix select: key T of the lp-th largest score and `need`
  // three digits of 11, 11 and 10 bits into one shared 2048-bin histogram;
  // thread t owns bins 2t and 2t+1, reads and clears them after the counts
  for (int b = tid; b < kSelBins; b += kRegThreads) hist[b] = 0u;
  __syncthreads();
  uint32_t prefix = 0u, prefix_mask = 0u, remaining = (uint32_t)lp;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
    const uint32_t dmask = pass == 2 ? 1023u : 2047u;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const uint32_t kj = key[j];
      if (j < n_valid && (kj & prefix_mask) == prefix) atomicAdd(&hist[(kj >> shift) & dmask], 1u);
    }
    __syncthreads();
    const uint32_t c0 = hist[2 * tid], c1 = hist[2 * tid + 1];
    hist[2 * tid] = 0u;
    hist[2 * tid + 1] = 0u;
    const uint32_t own = c0 + c1;
    const uint32_t pre = wave_prefix_sum(own);  // bins of the lanes <= lane
    const uint32_t wt = (uint32_t)__builtin_amdgcn_readlane((int)pre, 63);
    uint32_t incl = wt - pre + own;  // inclusive suffix sum over the lanes >= lane
    if (lane == 0) wtot[wave] = wt;
    __syncthreads();
#pragma unroll
    for (int w = 1; w < kRegWaves; ++w) incl += w > wave ? wtot[w] : 0u;
    const uint32_t above_t = incl - own;  // keys in the bins above 2t+1
    if (above_t < remaining && remaining <= incl) {
      if (remaining <= above_t + c1) {
        sel_digit = (uint32_t)(2 * tid + 1);
        sel_above = above_t;
      } else {
        sel_digit = (uint32_t)(2 * tid);
        sel_above = above_t + c1;
      }
    }
    __syncthreads();
    prefix |= sel_digit << shift;
    prefix_mask |= dmask << shift;
    remaining -= sel_above;
  }
  const uint32_t T = prefix;
  const uint32_t need = remaining;

  // ---- 2. counts above / equal to T before this thread's range (block scan)
  uint32_t n_gt = 0u, n_eq = 0u;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const uint32_t kj = key[j];
    n_gt += (j < n_valid && kj > T) ? 1u : 0u;
    n_eq += (j < n_valid && kj == T) ? 1u : 0u;
  }
  const uint32_t x_gt = wave_prefix_sum(n_gt), x_eq = wave_prefix_sum(n_eq);  // inclusive
  if (lane == 63) { wsum_gt[wave] = x_gt; wsum_eq[wave] = x_eq; }
  __syncthreads();
  uint32_t gt_before = x_gt - n_gt, eq_before = x_eq - n_eq;
#pragma unroll
  for (int w = 0; w < kRegWaves - 1; ++w) {
    gt_before += w < wave ? wsum_gt[w] : 0u;
    eq_before += w < wave ? wsum_eq[w] : 0u;
  }

  // ---- 3. this workgroup's share of output positions: its list in LDS
  const int p0 = blockIdx.x * share, p1 = min(lp, p0 + share);
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const uint32_t kj = key[j];
    const bool gt = j < n_valid && kj > T;
    const bool eq = j < n_valid && kj == T;
    const uint32_t pos = gt_before + min(eq_before, need);
    const bool sel = gt || (eq && eq_before < need);
    if (sel && (int)pos >= p0 && (int)pos < p1) {
      list_src[pos - p0] = i0 + j;
      if (out_idx) out_idx[(size_t)head * lp + pos] = i0 + j;
    }
    gt_before += gt ? 1u : 0u;
    eq_before += eq ? 1u : 0u;
  }
  __syncthreads();

  // ---- 4. gather the share's rows with 16-byte copies
  const int row_chunks = head_dim / 8;
  const size_t M = (size_t)La + Lb;
  const uint4* ksrc = reinterpret_cast<const uint4*>(k + (size_t)head * M * head_dim);
  const uint4* vsrc = reinterpret_cast<const uint4*>(v + (size_t)head * M * head_dim);
  uint4* kdst = reinterpret_cast<uint4*>(out_k + (size_t)head * lp * head_dim);
  uint4* vdst = reinterpret_cast<uint4*>(out_v + (size_t)head * lp * head_dim);
  const int pieces = (p1 - p0) * row_chunks;
  for (int e = tid; e < 2 * pieces; e += kRegThreads) {
    const int which = e >= pieces;  // 0: K, 1: V
    const int ee = e - which * pieces;
    const int r = ee / row_chunks, ch = ee - r * row_chunks;
    const int li = list_src[r];
    if (li < 0 || li >= Lb) continue;
    const size_t src = ((size_t)La + li) * row_chunks + ch;
    const size_t dst = (size_t)(p0 + r) * row_chunks + ch;
    if (which) vdst[dst] = vsrc[src];
    else kdst[dst] = ksrc[src];
  }
}

// ---------------------------------------------------------------------------
// Long local blocks (Lb > kRegMaxKeys): the scores are streamed from L2 instead
// of held, and the threshold's digits are not counted over all of them.  At
// 131072 power-law scores (l_p = 16384, 8 heads of d = 128) a call takes 73 us,
// of which the 139 MB it has to move take 27; radix passes over all scores by
// 256 threads had taken 655.  Bound by the one pass over the scores (its vector
// instructions: every workgroup of a head repeats it) and then the gather.
//  1. 4096 sample keys, one from every 4096th part of the block at a scattered
//     place in it, taken to 22 bits by two histogram passes, give a bracket [lo,
//     hi] that holds the l_p-th largest key but for a chance of 1e-4 (four
//     standard deviations of its sample rank to either side: 4% of the keys at
//     l_p = Lb / 8, 6.5% at Lb / 2).
//  2. One pass over the keys (16-byte loads, eight in flight per lane) counts
//     those above hi by ballot, per chunk of kLongBlock << m keys, and keeps
//     those inside the bracket, with their chunk, in LDS.  No atomics: scores
//     like N(0,1) put most keys of a wave into a few bins, and histogram
//     atomics on one bin take a turn each.
//     A bracket with far more sample keys in it than it was asked for has tied
//     groups at its ends, or scores that differ in their last 10 bits alone.  A
//     third histogram pass then makes lo and hi the sample's own keys, and the
//     pass counts the keys equal to either instead of keeping them: more
//     instructions per key, so for such blocks only (65536 scores, 8 heads: N(0,1)
//     37 us; 1 + 1e-5 N(0,1) 50, where the kept keys overflow without it 128; one
//     value alone 64 against 123).
//  3. A radix select of the kept keys, relative to lo, gives the threshold.
//     When the bracket misses it or more keys fall inside than LDS holds (past
//     250 000 to 380 000 rows: 6.5 or 4% of them; the pass is left out where the
//     sample says so), a radix select over all keys takes its place.
//  4. A scan over the chunks gives every chunk its output position; the
//     workgroup reads again only the chunks its share of the output positions
//     touches, lists their selected rows and gathers them.
// Same threshold, tie rule and output as the register form.
constexpr int kLongBlock = 256;      // keys a wave takes at a time (one float4 per lane)
constexpr int kLongChunks = 1024;    // chunks of a head, one per thread in the scan
constexpr int kLongCap = 1024;       // bracket keys a wave keeps
constexpr int kLongBatch = 8;        // blocks a wave loads ahead
constexpr int kLongSample = 4096;
constexpr int kLongList = 1024;      // output rows listed at a time

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct LongShared {
  uint32_t hist[2][kSelBins];
  u32x2 cand[kRegWaves][kLongCap];  // score, chunk
  uint32_t gt[kLongChunks + 1], eq[kLongChunks + 1];
  int32_t list_src[kLongList];
  uint16_t hits[kLongChunks];
  uint32_t wtot[4][kRegWaves];
  uint32_t sel_digit[2], sel_above[2], sel_count[2];
  uint32_t n_hits, overflow;
};

// Of the 2048 bins of hist[0] and hist[1], the bin holding the rank[u]-th
// largest key of histogram u, the keys above that bin and in it; the bins are
// cleared.  Every thread calls it with all counts made (no barrier between).
__device__ __forceinline__ void find_bins(LongShared& sh, const uint32_t (&rank)[2],
                                          uint32_t (&digit)[2], uint32_t (&above)[2],
                                          uint32_t (&in)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();
  uint32_t c1[2], own[2], incl[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t c0 = sh.hist[u][2 * tid];
    c1[u] = sh.hist[u][2 * tid + 1];
    sh.hist[u][2 * tid] = 0u;
    sh.hist[u][2 * tid + 1] = 0u;
    own[u] = c0 + c1[u];
    const uint32_t pre = wave_prefix_sum(own[u]);
    const uint32_t wt = (uint32_t)__builtin_amdgcn_readlane((int)pre, 63);
    incl[u] = wt - pre + own[u];  // suffix sum over the lanes >= lane
    if (lane == 0) sh.wtot[u][wave] = wt;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int w = 1; w < kRegWaves; ++w) incl[u] += w > wave ? sh.wtot[u][w] : 0u;
    const uint32_t above_t = incl[u] - own[u];  // keys in the bins above 2t+1
    if (above_t < rank[u] && rank[u] <= incl[u]) {
      const bool upper = rank[u] <= above_t + c1[u];
      sh.sel_digit[u] = (uint32_t)(2 * tid) + (upper ? 1u : 0u);
      sh.sel_above[u] = above_t + (upper ? 0u : c1[u]);
      sh.sel_count[u] = upper ? c1[u] : own[u] - c1[u];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    digit[u] = sh.sel_digit[u];
    above[u] = sh.sel_above[u];
    in[u] = sh.sel_count[u];
  }
}

// The four scores of this lane in block b of nb (indices kLongBlock * b + 4 * lane
// ..); past the end +0 (such keys are never counted).
__device__ __forceinline__ f32x4 load_block(const float* s, int b, int nb, int Lb, bool vec) {
  const int lane = threadIdx.x & 63;
  f32x4 f = {0.f, 0.f, 0.f, 0.f};
  if (b < nb) {
    const int i0 = b * kLongBlock + 4 * lane, left = Lb - i0;
    if (vec && left >= 4) {
      f = *reinterpret_cast<const f32x4*>(s + i0);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < left) f[j] = s[i0 + j];
    }
  }
  return f;
}

// Calls body(block, scores, valid) for every block of this wave (wave, wave +
// 16, ...), with this lane's four scores, of which the first `valid` count;
// kLongBatch blocks' loads at a time and the next batch's in flight behind them.
template <typename Body>
__device__ __forceinline__ void for_blocks(const float* s, int Lb, Body body) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (Lb + kLongBlock - 1) / kLongBlock;
  const bool vec = ((uintptr_t)s & 15u) == 0;
  f32x4 next[kLongBatch];
#pragma unroll
  for (int u = 0; u < kLongBatch; ++u) next[u] = load_block(s, wave + kRegWaves * u, nb, Lb, vec);
  for (int b0 = wave; b0 < nb; b0 += kRegWaves * kLongBatch) {
    f32x4 cur[kLongBatch];
#pragma unroll
    for (int u = 0; u < kLongBatch; ++u) {
      cur[u] = next[u];
      next[u] = load_block(s, b0 + kRegWaves * (kLongBatch + u), nb, Lb, vec);
    }
#pragma unroll
    for (int u = 0; u < kLongBatch; ++u) {
      const int b = b0 + kRegWaves * u;
      if (b < nb) body(b, cur[u], Lb - (b * kLongBlock + 4 * lane));
    }
  }
}

__global__ void __launch_bounds__(kRegThreads)
topk_gather_long_kernel(const float* __restrict__ scores, const uint16_t* __restrict__ k,
                        const uint16_t* __restrict__ v, int32_t* __restrict__ out_idx,
                        uint16_t* __restrict__ out_k, uint16_t* __restrict__ out_v, int La,
                        int Lb, int lp, int n_kv, int head_dim, int share, int chunk_shift) {
  __shared__ LongShared sh;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive workgroups go to different XCDs: with n_kv = 8 a head's scores
  // stay in one L2
  const int head = blockIdx.x % n_kv;
  const float* s = scores + (size_t)head * Lb;
  const int nb = (Lb + kLongBlock - 1) / kLongBlock;
  const int nchunks = ((nb - 1) >> chunk_shift) + 1;

  for (int i = tid; i < 2 * kSelBins; i += kRegThreads) (&sh.hist[0][0])[i] = 0u;
  for (int i = tid; i <= kLongChunks; i += kRegThreads) sh.gt[i] = sh.eq[i] = 0u;
  if (tid == 0) sh.overflow = 0u;

  // ---- 1. the bracket, from the sample.  Its places are scattered (multiples of
  // 2^32 / golden ratio): evenly spaced ones could follow a pattern of the scores
  uint32_t smp[kLongSample / kRegThreads];
#pragma unroll
  for (int j = 0; j < kLongSample / kRegThreads; ++j) {
    const uint32_t i = (uint32_t)(j * kRegThreads + tid), part = (uint32_t)Lb / kLongSample;
    const uint32_t from = i * part + i * ((uint32_t)Lb % kLongSample) / kLongSample;
    smp[j] = score_key(s[from + __umulhi(i * 0x9e3779b9u, part)]);
  }
  __syncthreads();
  const float mean = (float)lp / (float)Lb * kLongSample;
  const float dev = 4.f * sqrtf(fmaxf(mean * (1.f - mean / kLongSample), 0.f)) + 4.f;
  uint32_t rank[2] = {(uint32_t)max(1, (int)(mean - dev)),
                      (uint32_t)min(kLongSample, (int)(mean + dev) + 1)};
  uint32_t digit[2], above[2], in[2], top[2];
  const uint32_t first_rank = rank[0], last_rank = rank[1];
  const bool open_hi = first_rank <= 1, open_lo = last_rank >= kLongSample;
#pragma unroll
  for (int j = 0; j < kLongSample / kRegThreads; ++j) {
    atomicAdd(&sh.hist[0][smp[j] >> 21], 1u);
    atomicAdd(&sh.hist[1][smp[j] >> 21], 1u);
  }
  find_bins(sh, rank, digit, above, in);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    top[u] = digit[u];
    rank[u] -= above[u];
  }
#pragma unroll
  for (int j = 0; j < kLongSample / kRegThreads; ++j)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (smp[j] >> 21 == top[u]) atomicAdd(&sh.hist[u][(smp[j] >> 10) & 2047u], 1u);
  find_bins(sh, rank, digit, above, in);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    top[u] = top[u] << 11 | digit[u];
    rank[u] -= above[u];
  }
  // to 22 bits: the upper edge of hi's bin, the lower edge of lo's; an end of
  // the sample leaves its side open
  uint32_t hi = open_hi ? 0xffffffffu : (top[0] << 10 | 1023u);
  uint32_t lo = open_lo ? 0u : top[1] << 10;
  // sample keys in the bracket, and as many as it was asked for
  const uint32_t asked = last_rank - first_rank + 1;
  uint32_t inside = (open_lo ? (uint32_t)kLongSample : last_rank - rank[1] + in[1]) -
                    (open_hi ? 0u : first_rank - rank[0]);
  const bool exact = inside > 2 * asked;
  if (exact) {
#pragma unroll
    for (int j = 0; j < kLongSample / kRegThreads; ++j)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (smp[j] >> 10 == top[u]) atomicAdd(&sh.hist[u][smp[j] & 1023u], 1u);
    find_bins(sh, rank, digit, above, in);
    if (!open_hi) hi = top[0] << 10 | digit[0];
    if (!open_lo) lo = top[1] << 10 | digit[1];
    inside = asked;  // at most, between lo and hi
  }

  // The pass compares the scores themselves, which agrees with the keys once
  // no bound lies between -0 and +0 or between NaN and -inf (NaN compares
  // false with all, so it is neither above nor inside; if the threshold is
  // down there, the counts below say so).
  const bool in_nan = hi < 0x007fffffu;  // a threshold that only the keys order
  if (hi == 0x7fffffffu) hi = 0x80000000u;
  hi = max(hi, 0x007fffffu);
  lo = max(lo, 0x007fffffu);
  const float hi_f = key_score(hi), lo_f = key_score(lo);
  const bool pass = !in_nan && (float)inside * ((float)Lb / kLongSample) <
                                   1.1f * (float)(kLongCap * kRegWaves);

  // ---- 2. one pass: keys above hi per chunk, bracket keys kept; if exact,
  // those equal to hi (hist[1]) and to lo (eq) per chunk instead
  uint32_t kept = 0u;  // this wave's bracket keys
  auto keep = [&](unsigned long long m, float f, uint32_t chunk) __attribute__((always_inline)) {
    const uint32_t at = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, kept));
    // (m as the lanes' condition: testing m >> lane & 1 took three vector
    // instructions more per 64 keys; 131072 power-law scores, inputs rotating,
    // 75.9 -> 74.0 us)
    if (__builtin_amdgcn_inverse_ballot_w64(m) && at < (uint32_t)kLongCap)
      sh.cand[wave][at] = u32x2{__float_as_uint(f), chunk};
    kept += (uint32_t)__popcll(m);
  };
  if (pass && !exact) {
    for_blocks(s, Lb, [&](int b, f32x4 f, int valid) __attribute__((always_inline)) {
      const uint32_t chunk = (uint32_t)(b >> chunk_shift);
      const bool full = (b + 1) * kLongBlock <= Lb;
      uint32_t n_gt = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned long long above_m = __ballot(f[j] > hi_f), m = __ballot(f[j] >= lo_f);
        if (!full) {
          const unsigned long long ok = __ballot(j < valid);
          above_m &= ok;
          m &= ok;
        }
        n_gt += (uint32_t)__popcll(above_m);
        keep(m & ~above_m, f[j], chunk);
      }
      if (lane == 0 && n_gt) atomicAdd(&sh.gt[chunk], n_gt);
    });
  } else if (pass) {
    for_blocks(s, Lb, [&](int b, f32x4 f, int valid) __attribute__((always_inline)) {
      const uint32_t chunk = (uint32_t)(b >> chunk_shift);
      uint32_t n_gt = 0u, n_hi = 0u, n_lo = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned long long ok = __ballot(j < valid);
        const unsigned long long gt_hi = __ballot(f[j] > hi_f) & ok, ge_hi = __ballot(f[j] >= hi_f) & ok;
        const unsigned long long gt_lo = __ballot(f[j] > lo_f) & ok, ge_lo = __ballot(f[j] >= lo_f) & ok;
        n_gt += (uint32_t)__popcll(gt_hi);
        n_hi += (uint32_t)__popcll(ge_hi & ~gt_hi);
        n_lo += (uint32_t)__popcll(ge_lo & ~gt_lo);
        keep(gt_lo & ~ge_hi, f[j], chunk);  // (an open hi compares false)
      }
      if (lane == 0) {
        if (n_gt) atomicAdd(&sh.gt[chunk], n_gt);
        if (n_hi) atomicAdd(&sh.hist[1][chunk], n_hi);
        if (n_lo) atomicAdd(&sh.eq[chunk], n_lo);
      }
    });
  }
  if (lane == 0) {
    sh.wtot[0][wave] = kept;
    if (kept > (uint32_t)kLongCap) sh.overflow = 1u;
  }
  __syncthreads();
  // this thread's chunk (kLongChunks == kRegThreads); one key alone is hi
  const uint32_t my_gt = sh.gt[tid];
  uint32_t my_hi = 0u, my_lo = 0u;
  const bool overflow = sh.overflow != 0u;
  {
    const uint32_t g = wave_prefix_sum(my_gt);
    if (lane == 63) sh.wtot[1][wave] = g;
  }
  if (exact) {
    my_hi = sh.hist[1][tid];
    my_lo = lo == hi ? 0u : sh.eq[tid];
    sh.hist[1][tid] = 0u;
    const uint32_t h = wave_prefix_sum(my_hi), l = wave_prefix_sum(my_lo);
    if (lane == 63) {
      sh.wtot[2][wave] = h;
      sh.wtot[3][wave] = l;
    }
  }
  __syncthreads();
  uint32_t n_in = 0u, n_above = 0u, n_hi = 0u, n_lo = 0u;
  for (int w = 0; w < kRegWaves; ++w) {
    n_in += sh.wtot[0][w];
    n_above += sh.wtot[1][w];
  }
  if (exact) {
    for (int w = 0; w < kRegWaves; ++w) {
      n_hi += sh.wtot[2][w];
      n_lo += sh.wtot[3][w];
    }
  }

  // ---- 3. threshold key T and how many of the keys equal to it are selected
  // (from the pass: hi, a kept key or lo)
  const bool kept_all = pass && !overflow && n_above < (uint32_t)lp &&
                        (uint32_t)lp <= n_above + n_hi + n_in + n_lo;
  const bool at_hi = kept_all && (uint32_t)lp <= n_above + n_hi;
  const bool at_lo = kept_all && (uint32_t)lp > n_above + n_hi + n_in;
  uint32_t remaining = (uint32_t)lp;
  if (kept_all) {
    remaining -= n_above + (at_hi ? 0u : n_hi) + (at_lo ? n_in : 0u);
    sh.gt[tid] = my_gt + (at_hi ? 0u : my_hi);
    sh.eq[tid] = at_hi ? my_hi : at_lo ? my_lo : 0u;
  } else {
    lo = 0u;
    hi = 0xffffffffu;
    sh.gt[tid] = sh.eq[tid] = 0u;
  }
  int bits = at_hi || at_lo || lo == hi ? 0 : 32 - __builtin_clz(hi - lo);
  uint32_t prefix = at_hi ? hi - lo : 0u;  // of key - lo, its bits from `bits` up
  const uint32_t mine = min(kept, (uint32_t)kLongCap);
  while (bits > 0) {
    const int w = min(11, bits), above_bits = bits;
    bits -= w;
    // (A shift by 32 is not defined; then every key counts.)  With ties, the
    // lanes of a wave that share the first lane's bin, then those that share the
    // next one's, add together: their atomics would take a turn each.
    auto count = [&](uint32_t d, bool valid, auto ties) __attribute__((always_inline)) {
      const uint32_t bin = d >> bits & ((1u << w) - 1u);
      unsigned long long todo = __ballot(valid && (above_bits == 32 || d >> above_bits == prefix));
#pragma unroll
      for (int round = 0; round < (decltype(ties)::value ? 2 : 0); ++round) {
        if (todo == 0) break;
        const int leader = __builtin_ctzll(todo);
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
        const unsigned long long same = __ballot(bin == first) & todo;
        if (lane == leader) atomicAdd(&sh.hist[0][first], (uint32_t)__popcll(same));
        todo &= ~same;
      }
      if (todo >> lane & 1) atomicAdd(&sh.hist[0][bin], 1u);
    };
    auto count_kept = [&](auto ties) __attribute__((always_inline)) {
      for (uint32_t i = 0; i < mine; i += 64) {
        const bool valid = i + lane < mine;
        count(valid ? score_key(__uint_as_float(sh.cand[wave][i + lane][0])) - lo : 0u, valid, ties);
      }
    };
    if (kept_all && n_in <= (uint32_t)Lb / 8) {  // the bracket alone holds about 4%
      count_kept(std::false_type{});
    } else if (kept_all) {
      count_kept(std::true_type{});
    } else {
      for_blocks(s, Lb, [&](int, f32x4 f, int valid) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) count(score_key(f[j]) - lo, j < valid, std::true_type{});
      });
    }
    rank[0] = remaining;
    rank[1] = 0u;  // unused: no bin matches
    find_bins(sh, rank, digit, above, in);
    prefix = prefix << w | digit[0];
    remaining -= above[0];
  }
  const uint32_t T = lo + prefix;
  const uint32_t need = remaining;

  // ---- 4. keys above and equal to T per chunk, then before every chunk
  __syncthreads();
  if (kept_all) {
    for (uint32_t i = lane; i < mine; i += 64) {
      const u32x2 c = sh.cand[wave][i];
      const uint32_t key = score_key(__uint_as_float(c[0]));
      if (key > T) atomicAdd(&sh.gt[c[1]], 1u);
      else if (key == T) atomicAdd(&sh.eq[c[1]], 1u);
    }
  } else {
    for_blocks(s, Lb, [&](int b, f32x4 f, int valid) __attribute__((always_inline)) {
      uint32_t n_gt = 0u, n_eq = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t key = score_key(f[j]);
        n_gt += (uint32_t)__popcll(__ballot(j < valid && key > T));
        n_eq += (uint32_t)__popcll(__ballot(j < valid && key == T));
      }
      if (lane == 0) {
        const uint32_t chunk = (uint32_t)(b >> chunk_shift);
        if (n_gt) atomicAdd(&sh.gt[chunk], n_gt);
        if (n_eq) atomicAdd(&sh.eq[chunk], n_eq);
      }
    });
  }
  __syncthreads();
  {
    const uint32_t g = sh.gt[tid], e = sh.eq[tid];
    uint32_t xg = wave_prefix_sum(g), xe = wave_prefix_sum(e);
    if (lane == 63) {
      sh.wtot[0][wave] = xg;
      sh.wtot[1][wave] = xe;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kRegWaves - 1; ++w) {
      xg += w < wave ? sh.wtot[0][w] : 0u;
      xe += w < wave ? sh.wtot[1][w] : 0u;
    }
    sh.gt[tid + 1] = xg;  // element 0 stays 0 below
    sh.eq[tid + 1] = xe;
    if (tid == 0) sh.gt[0] = sh.eq[0] = 0u;
  }

  // ---- 5. this workgroup's share of the output positions, a list at a time
  const int p_begin = (int)(blockIdx.x / n_kv) * share, p_end = min(lp, p_begin + share);
  const int row_chunks = head_dim / 8;  // 16-byte pieces per row
  const size_t M = (size_t)La + Lb;
  const u32x4* ksrc = reinterpret_cast<const u32x4*>(k + (size_t)head * M * head_dim);
  const u32x4* vsrc = reinterpret_cast<const u32x4*>(v + (size_t)head * M * head_dim);
  u32x4* kdst = reinterpret_cast<u32x4*>(out_k + (size_t)head * lp * head_dim);
  u32x4* vdst = reinterpret_cast<u32x4*>(out_v + (size_t)head * lp * head_dim);
  for (int p0 = p_begin; p0 < p_end; p0 += kLongList) {
    const int p1 = min(p_end, p0 + kLongList);
    if (tid == 0) sh.n_hits = 0u;
    // every slot is filled below (exactly lp positions are selected); -1
    // marks a slot as empty for the gather regardless
    sh.list_src[tid] = -1;
    __syncthreads();
    if (tid < nchunks) {
      const uint32_t first = sh.gt[tid] + min(sh.eq[tid], need);
      const uint32_t last = sh.gt[tid + 1] + min(sh.eq[tid + 1], need);
      if (first < (uint32_t)p1 && last > (uint32_t)p0 && first < last)
        sh.hits[atomicAdd(&sh.n_hits, 1u)] = (uint16_t)tid;
    }
    __syncthreads();
    const int n_hits = (int)sh.n_hits;
    for (int h = wave; h < n_hits; h += kRegWaves) {
      const int chunk = sh.hits[h];
      uint32_t n_gt = sh.gt[chunk], n_eq = sh.eq[chunk];
      const int c0 = (chunk << chunk_shift) * kLongBlock;
      const int c1 = min(Lb, c0 + (kLongBlock << chunk_shift));
      for (int base = c0; base < c1; base += 4 * 64) {
        float f[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = base + 64 * j + lane < c1 ? s[base + 64 * j + lane] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = base + 64 * j + lane;
          const uint32_t key = score_key(f[j]);
          const unsigned long long mg = __ballot(i < c1 && key > T);
          const unsigned long long me = __ballot(i < c1 && key == T);
          const bool gt = i < c1 && key > T, eq = i < c1 && key == T;
          const uint32_t rg = n_gt + __builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0u));
          const uint32_t re = n_eq + __builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0u));
          const uint32_t pos = rg + min(re, need);
          if ((gt || (eq && re < need)) && pos >= (uint32_t)p0 && pos < (uint32_t)p1) {
            sh.list_src[pos - p0] = i;
            if (out_idx) out_idx[(size_t)head * lp + pos] = i;
          }
          n_gt += (uint32_t)__popcll(mg);
          n_eq += (uint32_t)__popcll(me);
        }
      }
    }
    __syncthreads();
    const int pieces = (p1 - p0) * row_chunks;  // per tensor
    for (int e = tid; e < pieces; e += kRegThreads) {
      const int r = e / row_chunks, ch = e - r * row_chunks;
      const int li = sh.list_src[r];
      if (li < 0 || li >= Lb) continue;
      const size_t src = ((size_t)La + li) * row_chunks + ch;
      const size_t dst = (size_t)(p0 + r) * row_chunks + ch;
      const u32x4 kx = ksrc[src], vx = vsrc[src];
      kdst[dst] = kx;
      vdst[dst] = vx;
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_compress(const CompressArgs& a, hipStream_t stream) {
  if (a.lp == 0) return hipSuccess;
  if (a.Lb <= kRegMaxKeys) {
    // a share of at most 1024 output rows per workgroup, about 64 rows each
    // for the gather, at most 32 workgroups per head
    int groups = (a.lp + 63) / 64;
    groups = groups < 1 ? 1 : (groups > 32 ? 32 : groups);
    int share = (a.lp + groups - 1) / groups;
    if (share > 1024) {
      share = 1024;
      groups = (a.lp + share - 1) / share;
    }
    const dim3 grid(groups, a.n_kv);
    if (a.Lb <= kRegThreads * 4)
      hipLaunchKernelGGL(topk_gather_reg_kernel<4>, grid, dim3(kRegThreads), 0, stream, a.scores,
                         a.k, a.v, a.idx, a.out_k, a.out_v, a.La, a.Lb, a.lp, a.head_dim, share);
    else
      hipLaunchKernelGGL(topk_gather_reg_kernel<16>, grid, dim3(kRegThreads), 0, stream, a.scores,
                         a.k, a.v, a.idx, a.out_k, a.out_v, a.La, a.Lb, a.lp, a.head_dim, share);
    return hipGetLastError();
  }
  // about 64 rows or more per workgroup for the gather, at most a workgroup per
  // CU over all heads (a head's workgroups each repeat its select); below 32
  // workgroups 16 rows or more, few selected rows being spread over as many chunks
  // to read again (20000 scores, 8 heads, l_p = 64: 21.2 -> 18.1 us)
  int groups = std::max(a.lp / 64 + (a.lp % 64 != 0), std::min(32, a.lp / 16 + (a.lp % 16 != 0)));
  groups = std::min(groups, std::max(1, 256 / a.n_kv));
  const int share = a.lp / groups + (a.lp % groups != 0);
  const int blocks = (a.Lb + kLongBlock - 1) / kLongBlock;
  int chunk_shift = 0;
  while (((blocks - 1) >> chunk_shift) >= kLongChunks) ++chunk_shift;
  hipLaunchKernelGGL(topk_gather_long_kernel, dim3((unsigned)(groups * a.n_kv)), dim3(kRegThreads), 0,
                     stream, a.scores, a.k, a.v, a.idx, a.out_k, a.out_v, a.La, a.Lb, a.lp, a.n_kv,
                     a.head_dim, share, chunk_shift);
  return hipGetLastError();
}

}  // namespace apb
