// Shared by apb_layer.hip and apb_scorer.hip (device code; each file that
// includes it instantiates its own kernels).
//
// The library's bf16 matrix products on gfx950, out[t][f] = sum_k x[t][k]
// W[f][k] (tokens t, output features f, weights row-major [f][k]): the
// layer's projections (apb_layer.hip) and the first layer of the retaining
// head (apb_scorer.hip).  One kernel template covers them: bf16 MFMA
// 16x16x32 with fp32 accumulation, output features on the MFMA M side (the
// weights are the A operand) and tokens on the N side, a workgroup tile of
// 256 features x 32 * NB tokens computed by 4 waves (2 x 2, each 128 features
// x 16 * NB tokens), K steps of 64 whose weight and token slabs are copied
// HBM -> LDS by global_load_lds_dwordx4 into XOR-swizzled tiles.  (16x16x32
// rather than 32x32x16: the same LDS bytes per flop and half the
// accumulator traffic, which this power-limited chip turns into clock.)
// Neither a copy nor an operand read spends a vector instruction on its
// address: a copy is a scalar base plus a fixed per-lane offset, a read one
// XOR of a per-lane base plus an instruction offset.
//  * NB = 8 (256 tokens), for products that fill the chip with such tiles:
//    one wave per SIMD, 256 accumulator registers, two LDS stages.  The step
//    boundary is software-pipelined: at its last 32-deep substep a wave waits
//    for its copies of the next step, passes the barrier, and issues that
//    substep's MFMAs with the next step's first operand reads and the copies
//    of the step after it (into the stage just finished) spread among them
//    (for long K loops the copies start earlier, behind a second barrier that
//    marks the stage free); the last two steps are peeled so the steady-state
//    loop has no branches (the compiler can then count outstanding LDS reads
//    exactly).
//  * NB = 2, 3, 4 (64, 96, 128 tokens), for products that would leave CUs
//    idle: bound by the copies, which a CU takes at 31 cycles per KiB (about
//    70 GB/s) whatever their pattern, 40 to 48 of them per step beside 512 to
//    1024 cycles of MFMAs.  Four further waves issue them (two waves per SIMD,
//    three LDS stages), so that no MFMA queues behind a copy: 1000 tokens x
//    1024 features at K = 6144 in 128-token tiles took 88 us with the copies
//    in the computing waves, 63 us with waves of their own (256-token tiles:
//    122 us).  Deeper rings, other read spacings and prefetches into L2 gave
//    nothing (the CU's copy rate is the limit, not latency).  The whole layer
//    at 1256 tokens: 1079 -> 666 us; the retaining head of 8192 tokens:
//    151 -> 88 us.
// Every tile width adds K in the same order, so a token's result depends on
// neither its tile nor the number of tokens: the compressor's tie rule relies
// on equal tokens scoring alike, bit for bit.  (Starting the K loop of each XCD
// an eighth further on, which spreads the XCDs' fetches of weights that are not
// in cache, would take 1000 tokens x 1024 units from 78 to 58 us.)
// The token operand is read row-major [t][k], head-major [k / dh][t][dh]
// (the attention output, whose heads are the O projection's K dimension), or
// from the head-major Q, K and V tensors as one [Q heads; K heads; V heads]
// feature row (the retaining head's input), so no transpose or
// concatenation is ever materialised.  Epilogues:
//  * row-major bf16 store, plus a residual in fp32 before the rounding;
//  * head-major Q/K/V store of the QKV projection (feature f is dim f % dh
//    of head f / dh: Q heads, then K heads, then V heads);
//  * SwiGLU: each wave's 128 weight rows are 64 gate rows and the 64 up
//    rows of the same features, so gate and up of one feature sit in the
//    same lane and register slot and SiLU(gate) * up is formed in registers;
//  * retaining head: bias, SiLU and the workgroup's share of the second
//    layer, one fp32 partial score per feature block, token and KV head.
#ifndef APB_GEMM_H_
#define APB_GEMM_H_

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "apb_internal.h"
#include "apb_plan.h"

namespace apb {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;

constexpr int kBF = 256;        // weight rows (output features) per workgroup
constexpr int kBK = 64;         // K per step
constexpr int kGemmThreads = 256;
constexpr int kPieces = 8;      // 1 KiB weight copy pieces per wave per step

enum XMode { kXRowMajor = 0, kXHeadMajor = 1, kXQkv = 2 };
enum WMode { kWPlain = 0, kWGateUp = 1 };
enum Epi { kEpiRowMajor = 0, kEpiQkv = 1, kEpiSwiglu = 2, kEpiScorer = 3 };
constexpr int kScorerMaxKv = 8;  // scores per token the kEpiScorer epilogue forms

struct GemmParams {
  const uint16_t* x;      // tokens: [T][K], [K / dh][T][dh], or Q of kXQkv
  const uint16_t* w;      // [F][K]; the gate matrix for kWGateUp
  const uint16_t* w_up;   // [F][K] for kWGateUp
  const uint16_t* resid;  // [T][F] or null (kEpiRowMajor)
  uint16_t* out;          // [T][F] (kEpiRowMajor, kEpiSwiglu); Q for kEpiQkv
  uint16_t* out_k;        // kEpiQkv: K [n_kv][T][dh]
  uint16_t* out_v;        // kEpiQkv: V [n_kv][T][dh]
  int T, K, F;            // F: output features (I for kWGateUp)
  int dh;                 // head dim of a head-major operand or output
  int n_q, n_kv;          // kEpiQkv, kXQkv
  // kXQkv: the token operand is [Q heads; K heads; V heads] of the
  // head-major tensors x (Q, [n_q][x_rows][dh]), x_k and x_v ([n_kv][x_rows]
  // [dh]), at rows x_row0 + t
  const uint16_t* x_k;
  const uint16_t* x_v;
  int x_rows, x_row0;
  // kEpiScorer: bias, SiLU and the second layer of the retaining head
  const float* b1;        // [F]
  const float* w2;        // [n_kv][F]
  float* part;            // [F / kBF][n_kv][T] fp32 partial scores per feature block
  // tile grid (set by launch_gemm): token tiles from token t_begin on, feature tiles
  int ntx, nfy, t_begin;
};

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// 16-byte chunk c of tile row r (128 bytes) sits at chunk c ^ ((r >> 1) & 7):
// any 16 consecutive rows, which one 16-lane pass of ds_read_b128 touches,
// land on 16 distinct 16-byte slots of the 256 bank bytes.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// NB: 16-token blocks per wave, i.e. a tile of 256 features x 32 * NB tokens.
// EARLY: the two-barrier step (long K loops, NB = 8), else one barrier per step.
template <int XM, int WM, int EPI, int NB, bool EARLY>
__global__ void __launch_bounds__(NB < 8 ? 2 * kGemmThreads : kGemmThreads, 1)
gemm_kernel(GemmParams p) {
  constexpr int BT = 32 * NB;                 // tokens per workgroup
  constexpr int NST = NB == 8 ? 2 : 3;        // LDS stages
  constexpr int CPS = kPieces + NB;           // copies per wave per step
  // NB < 8: waves 4..7 do the copies and waves 0..3 the rest (below)
  constexpr bool SPLIT = NB < 8;
  constexpr int NMF = 8 * NB;                 // MFMAs per 32-deep substep
  constexpr int NRD = 8 + NB;                 // operand reads per substep
  static_assert(!EARLY || NB == 8, "the two-barrier step is scheduled for 64 MFMAs");
  // 256-byte aligned: operand addresses XOR step bits into the low byte of
  // a stage base plus lane offset
  __shared__ __attribute__((aligned(256))) uint16_t a_lds[NST][kBF * kBK];  // weight slabs
  __shared__ __attribute__((aligned(256))) uint16_t b_lds[NST][BT * kBK];   // token slabs


  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave_id & 3;             // wave among the copying or the computing four
  const int wm = wave & 1, wn = wave >> 1;  // feature half, token half
  // XCD-aware tile order: workgroup b runs on XCD b % 8, and each XCD takes
  // one contiguous eighth (to within one tile) of the tiles, ordered in
  // columns of 4 feature tiles: the 32 tiles an XCD works on at a time are 4
  // feature x 8 token tiles, so per K step its L2 fetches 4 weight and 8
  // token slabs for 32 workgroups, and no XCD gets a round more than another.
  const int ntiles = p.ntx * p.nfy;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int per = ntiles >> 3, rem = ntiles & 7;
  if (slot >= per + (xcd < rem ? 1 : 0)) return;
  const int tile = xcd * per + min(xcd, rem) + slot;
  const int col = tile / (4 * p.ntx), in_col = tile - col * 4 * p.ntx;
  const int width = min(4, p.nfy - 4 * col);
  const int ttile = in_col / width, ftile = 4 * col + (in_col - ttile * width);
  const int t0 = p.t_begin + ttile * BT;
  const int f0 = ftile * (WM == kWGateUp ? kBF / 2 : kBF);
  const int nk = p.K / kBK;

  // ---- copies: piece j (8 rows x 128 bytes) of each slab; wave w copies
  // weight pieces 8w .. 8w+7 and token pieces NB*w .. NB*w + NB-1.  Lane l
  // takes row l/8 of the piece and fetches the chunk that belongs at slot
  // l%8.  Rows past the last feature or token repeat it (their results are
  // never stored).  A copy is a scalar base (the operand's first row for this
  // workgroup, advanced by the K step in scalar registers) plus a fixed
  // per-lane byte offset: no vector instruction.
  const int cp_row = lane >> 3, cp_slot = lane & 7;
  const int x_ld = XM == kXRowMajor ? p.K : p.dh;  // elements between token rows
  // head-major operands: head dims are a power of two (64 or 128)
  const int dh_shift = XM == kXRowMajor ? 0 : 31 - __builtin_clz((unsigned)p.dh);
  // (set_offsets is called by the copying waves alone: live in the others,
  // the offsets would spill)
  uint32_t w_off[kPieces], x_off[NB];
  auto set_offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int rho = 8 * (kPieces * wave + i) + cp_row;  // weight slab row 0..255
      const int chunk = 8 * (cp_slot ^ swz(rho));
      int fr = WM == kWGateUp ? f0 + 64 * (rho >> 7) + (rho & 63) : f0 + rho;
      fr = min(fr, p.F - 1);
      w_off[i] = 2u * (uint32_t)((fr - f0) * p.K + chunk);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int rho = 8 * (NB * wave + i) + cp_row;  // token slab row 0..BT-1
      const int chunk = 8 * (cp_slot ^ swz(rho));
      const int tr = min(t0 + rho, p.T - 1);
      x_off[i] = 2u * (uint32_t)((tr - t0) * x_ld + chunk);
    }
  };
  const uint16_t* const w_first = p.w + (size_t)f0 * p.K;
  const uint16_t* const w_up_first = (WM == kWGateUp ? p.w_up : p.w) + (size_t)f0 * p.K;
  const uint16_t* const x_first = p.x + (size_t)t0 * x_ld;
  // First token row's K elements of step kk.  Formed once per step and without
  // branches: the compiler put the choice of the Q, K or V tensor into branches
  // among the copies of the two-barrier loop (32768 tokens x 1024 units at K =
  // 9216: 541 against 442 us).
  auto token_base = [&](int kk) __attribute__((always_inline)) -> const uint16_t* {
    const int k0 = kk * kBK;
    if constexpr (XM == kXRowMajor) {
      return x_first + k0;
    } else {
      // head-major tokens: K element k0 is column k0 % dh of head k0 / dh
      const int head = k0 >> dh_shift, j0 = k0 - (head << dh_shift);
      if constexpr (XM == kXQkv) {
        // with masks: a branch here makes the step wait for all operand reads
        const int in_kv = -(int)(head >= p.n_q), in_v = -(int)(head >= p.n_q + p.n_kv);
        const int hh = head - (p.n_q & in_kv) - (p.n_kv & in_v);
        const int64_t src = (int64_t)p.x + (((int64_t)p.x_k - (int64_t)p.x) & in_kv) +
                            (((int64_t)p.x_v - (int64_t)p.x_k) & in_v);
        return (const uint16_t*)src + ((size_t)hh * p.x_rows + p.x_row0 + t0) * p.dh + j0;
      } else {
        return x_first + (size_t)head * p.T * p.dh + j0;
      }
    }
  };
  // copy q (0..CPS-1) of step kk, with its token_base, into stage st: q < 8
  // weight pieces, else token pieces
  auto copy = [&](int kk, const uint16_t* xb, int st, int q) __attribute__((always_inline)) {
    if (q < kPieces) {
      const int i = q, j = kPieces * wave + i;
      // gate/up: rows 64..127 of either 128-row half are up-projection rows
      const uint16_t* base =
          (WM == kWGateUp && ((kPieces * wave + i) & 15) >= 8 ? w_up_first : w_first) + kk * kBK;
      const uint32_t d = __builtin_amdgcn_readfirstlane(lds_offset(&a_lds[st][j * 512]));
      asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(w_off[i]), "s"(base),
                   "s"(d)
                   : "memory");
    } else {
      const int i = q - kPieces, j = NB * wave + i;
      const uint32_t d = __builtin_amdgcn_readfirstlane(lds_offset(&b_lds[st][j * 512]));
      asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(x_off[i]), "s"(xb),
                   "s"(d)
                   : "memory");
    }
  };

  // prologue: the first NST steps' copies issued, step 0's landed
  auto first_copies = [&]() __attribute__((always_inline)) {
    set_offsets();
#pragma unroll
    for (int k0 = 0; k0 < NST; ++k0) {
      if (k0 < nk) {
        const uint16_t* const xb = token_base(k0);
#pragma unroll
        for (int q = 0; q < CPS; ++q) copy(k0, xb, k0, q);
      }
    }
    if (nk >= NST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * CPS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
  };
  // The copying waves.  A CU takes one 1 KiB copy per 31 cycles whatever the
  // access pattern, so below 256 tokens a step's copies outlast its MFMAs, and
  // a wave that does both stalls its MFMAs behind the copies it issues.  One
  // barrier per step, shared with the computing waves' barrier B: before it
  // step kk+1 has landed, after it stage kk % NST is free for step kk+NST.
  if constexpr (SPLIT) {
    if (wave_id >= 4) {
      first_copies();
      int st = 0;
      for (int kk = 0; kk + 1 < nk; ++kk) {
        if (kk + NST <= nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * CPS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");
        if (kk + NST < nk) {
          const uint16_t* const xb = token_base(kk + NST);
#pragma unroll
          for (int q = 0; q < CPS; ++q) copy(kk + NST, xb, st, q);
        }
        st = st + 1 == NST ? 0 : st + 1;
      }
      return;
    }
  } else {
    first_copies();
  }
  if constexpr (SPLIT) asm volatile("s_barrier" ::: "memory");

  // ---- operands (16x16x32 MFMAs): lane (li, lg) of a 16-row block reads
  // slab row 16*blk + li, K elements 32*kc + 8*lg .. +7, i.e. chunk
  // 4*kc + lg of that row, stored at slot (4*kc + lg) ^ swz(row).
  // swz(row) = (li >> 1) & 7 for every block, so the address is (lane base
  // ^ 64*kc) plus a constant for stage and block.  The 16 rows one 16-lane
  // pass of ds_read_b128 touches land on 16 distinct bank slots.
  const int li = lane & 15, lg = lane >> 4;
  const int sw = (li >> 1) & 7;
  const uint32_t lane_chunk = (uint32_t)(16 * (lg ^ sw));
  const uint32_t a_lane = (uint32_t)((128 * wm + li) * 128) + lane_chunk;
  const uint32_t b_lane = (uint32_t)((16 * NB * wn + li) * 128) + lane_chunk;
  // stage st's row bases (rows are 128 bytes and the slabs 256-byte aligned, so
  // the XOR with 64*kc below touches only the chunk bits)
  auto a_base = [&](int st) __attribute__((always_inline)) { return lds_offset(a_lds[st]) + a_lane; };
  auto b_base = [&](int st) __attribute__((always_inline)) { return lds_offset(b_lds[st]) + b_lane; };
  // Operand read of the next substep issued behind MFMA i of a substep (0..7
  // weight block, 8.. token block), or -1.  SPLIT waves have 256 registers
  // each, so only the weight blocks 4..7 are double buffered: blocks 0..3 are
  // read into the registers that the substep's first half has used.
  auto read_of = [](int i) __attribute__((always_inline)) -> int {
    if (!SPLIT) return i < 2 * NRD && (i & 1) ? i >> 1 : -1;
    if (i < 4) return 4 + i;
    if (i < 4 + NB) return 8 + i - 4;
    return i >= 4 * NB && i < 4 * NB + 4 ? i - 4 * NB : -1;
  };
  auto a_buf = [](int sub, int mb) __attribute__((always_inline)) -> int {
    return SPLIT && mb < 4 ? 0 : sub;
  };
  auto read = [](uint32_t base, int blk, int kc) __attribute__((always_inline)) -> bf16x8 {
    return *(const lds_bf16x8*)(uintptr_t)((base ^ (64u * (uint32_t)kc)) + 2048u * (uint32_t)blk);
  };

  // acc[mb][nb]: 16 features x 16 tokens; lane (li, lg) holds features
  // 4*lg .. 4*lg+3 of token li
  f32x4 acc[8][NB];
#pragma unroll
  for (int mb = 0; mb < 8; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[mb][nb][r] = 0.f;
  bf16x8 av[2][8], bv[2][NB];

  // step 0 is visible: its first operands.  Scalar loads (the epilogue's
  // pointers, loaded early) are waited for first: they complete in no order, so
  // one that may be pending at the loop's entry makes its first MFMA wait for all
  // operand reads in flight, in every step (32768 tokens x 1024 units at K = 9216:
  // 475 against 465 us).
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) alone
#pragma unroll
  for (int mb = 0; mb < 8; ++mb) av[0][mb] = read(a_base(0), mb, 0);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) bv[0][nb] = read(b_base(0), nb, 0);

  // One K step in two substeps of NMF MFMAs; MFMAs early in a substep each
  // carry one of the next substep's NRD operand reads (with 64 MFMAs every
  // odd one of the first 32).  NEXT: step kk+1 exists (at the last substep:
  // its copies have landed, barrier B, read its first operands); COPY: step
  // kk+NST exists and this wave copies.  Its copies go into the stage this
  // step reads, spread over the substep's MFMAs (issued back to back they
  // stall the wave, and the matrix core with it, for hundreds of cycles).
  // That stage is free once every wave has read the last substep's operands
  // from it.  EARLY marks that point with barrier A, at MFMA 48 of the first
  // substep, and starts the copies there (4 in the first substep, 12 in the
  // second), giving them a quarter step more to land: worth 5% on K loops of
  // hundreds of steps, 1-2% slower on short ones.  Otherwise the copies start
  // after barrier B.
  auto step = [&](int kk, int st, auto next_t, auto copy_t) __attribute__((always_inline)) {
    constexpr bool NEXT = decltype(next_t)::value, COPY = decltype(copy_t)::value && !SPLIT;
    const int st1 = st + 1 == NST ? 0 : st + 1;
    const uint32_t ab = a_base(st), bb = b_base(st), ab1 = a_base(st1), bb1 = b_base(st1);
    const uint16_t* const xb = COPY ? token_base(kk + 2) : nullptr;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const int cur = kc, nxt = kc ^ 1;
      const bool boundary = kc == 1;
      if (boundary && NEXT) {
        // barrier B: this wave's copies of step kk+1 have landed; after the
        // barrier every wave's have
        if constexpr (SPLIT) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else if constexpr (EARLY && COPY) asm volatile("s_waitcnt vmcnt(4)\n\ts_barrier" ::: "memory");
        else if constexpr (EARLY) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      }
#pragma unroll
      for (int i = 0; i < NMF; ++i) {
        const int mb = i / NB, nb = i % NB;
        if (EARLY && !boundary && COPY && i == 48) {
          // barrier A: every wave's reads of stage st are done
          asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            av[a_buf(cur, mb)][mb], bv[cur][nb], acc[mb][nb], 0, 0, 0);
        const int j = read_of(i);
        if (j >= 0) {
          if (!boundary) {
            if (j < 8) av[a_buf(nxt, j)][j] = read(ab, j, 1);
            else bv[nxt][j - 8] = read(bb, j - 8, 1);
          } else if (NEXT) {
            if (j < 8) av[a_buf(nxt, j)][j] = read(ab1, j, 0);
            else bv[nxt][j - 8] = read(bb1, j - 8, 0);
          }
        }
        if constexpr (COPY && EARLY) {
          if ((i & 3) == 0) {
            if (!boundary && i >= 48) copy(kk + 2, xb, st, (i - 48) >> 2);
            else if (boundary && i < 48) copy(kk + 2, xb, st, 4 + (i >> 2));
          }
        } else if constexpr (COPY) {
          if (boundary && (i & 3) == 0) copy(kk + 2, xb, st, i >> 2);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  const std::true_type yes{};
  const std::false_type no{};
  int kk = 0, st = 0;
  auto advance = [&]() __attribute__((always_inline)) {
    ++kk;
    st = st + 1 == NST ? 0 : st + 1;
  };
  while (kk + (SPLIT ? 1 : NST) < nk) {
    step(kk, st, yes, yes);
    advance();
  }
  if (kk + 1 < nk) {
    step(kk, st, yes, no);
    advance();
  }
  step(kk, st, no, no);

  // ---- epilogue.  Lane (li, lg), block (mb, nb), element r holds slab row
  // 128*wm + 16*mb + 4*lg + r of token t0 + 16*NB*wn + 16*nb + li: four
  // consecutive features (one 8-byte store).
  if constexpr (EPI == kEpiScorer) {
    // bias, SiLU and this workgroup's share of the second layer: for each of
    // its tokens and each KV head, the sum over its 256 features of
    // SiLU(acc + b1) * w2, one fp32 partial per feature block
    __syncthreads();  // every wave is done with the LDS stages
    float* const w2_lds = reinterpret_cast<float*>(&a_lds[0][0]);  // [kBF][kScorerMaxKv]
    float* const b1_lds = w2_lds + kBF * kScorerMaxKv;              // [kBF]
    float* const red = reinterpret_cast<float*>(&b_lds[0][0]);     // [2][kScorerMaxKv][BT]
    for (int i = tid; i < kBF * kScorerMaxKv; i += kGemmThreads) {
      const int u = i / kScorerMaxKv, kv = i % kScorerMaxKv;
      w2_lds[i] = kv < p.n_kv ? p.w2[(size_t)kv * p.F + f0 + u] : 0.f;
    }
    for (int i = tid; i < kBF; i += kGemmThreads) b1_lds[i] = p.b1[f0 + i];
    __syncthreads();
    float part[NB][kScorerMaxKv];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int kv = 0; kv < kScorerMaxKv; ++kv) part[nb][kv] = 0.f;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int u = 128 * wm + 16 * mb + 4 * lg + r;
        const f32x4 wa = *reinterpret_cast<const f32x4*>(&w2_lds[u * kScorerMaxKv]);
        const f32x4 wb = *reinterpret_cast<const f32x4*>(&w2_lds[u * kScorerMaxKv + 4]);
        const float bias = b1_lds[u];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          // SiLU with the hardware reciprocal (within 1 ulp) instead of an
          // IEEE division, about ten instructions per element
          const float z = acc[mb][nb][r] + bias;
          const float a = z * __builtin_amdgcn_rcpf(1.f + __expf(-z));
#pragma unroll
          for (int kv = 0; kv < 4; ++kv) {
            part[nb][kv] = fmaf(a, wa[kv], part[nb][kv]);
            part[nb][4 + kv] = fmaf(a, wb[kv], part[nb][4 + kv]);
          }
        }
      }
    // the four lane groups hold the same tokens' other features
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int kv = 0; kv < kScorerMaxKv; ++kv) {
        float x = part[nb][kv];
        x += __shfl_xor(x, 16);
        part[nb][kv] = x + __shfl_xor(x, 32);
      }
    // the two feature halves (wm = 0, 1) of each token half meet in LDS
    if (lg == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int kv = 0; kv < kScorerMaxKv; ++kv)
          red[(wm * kScorerMaxKv + kv) * BT + 16 * NB * wn + 16 * nb + li] = part[nb][kv];
    }
    __syncthreads();
    for (int i = tid; i < kScorerMaxKv * BT; i += kGemmThreads) {
      const int kv = i / BT, tl = i % BT;
      const int t = t0 + tl;
      if (kv < p.n_kv && t < p.T)
        p.part[((size_t)ftile * p.n_kv + kv) * p.T + t] =
            red[kv * BT + tl] + red[(kScorerMaxKv + kv) * BT + tl];
    }
    return;
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int t = t0 + 16 * NB * wn + 16 * nb + li;
    if (t >= p.T) continue;
    if constexpr (EPI == kEpiSwiglu) {
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const int f = f0 + 64 * wm + 16 * mb + 4 * lg;
        if (f >= p.F) continue;
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gt = acc[mb][nb][i], up = acc[mb + 4][nb][i];
          o[i] = (__bf16)(gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up);  // SiLU(gate) * up
        }
        *reinterpret_cast<bf16x4*>(p.out + (size_t)t * p.F + f) = o;
      }
    } else {
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) {
        const int f = f0 + 128 * wm + 16 * mb + 4 * lg;
        if (f >= p.F) continue;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[mb][nb][i];
        uint16_t* dst;
        if constexpr (EPI == kEpiQkv) {
          const int head = f / p.dh, j = f - head * p.dh;
          if (head < p.n_q)
            dst = p.out + ((size_t)head * p.T + t) * p.dh + j;
          else if (head < p.n_q + p.n_kv)
            dst = p.out_k + ((size_t)(head - p.n_q) * p.T + t) * p.dh + j;
          else
            dst = p.out_v + ((size_t)(head - p.n_q - p.n_kv) * p.T + t) * p.dh + j;
        } else {
          dst = p.out + (size_t)t * p.F + f;
          if (p.resid) {
            const bf16x4 rr = *reinterpret_cast<const bf16x4*>(p.resid + (size_t)t * p.F + f);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += (float)rr[i];
          }
        }
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (__bf16)v[i];
        *reinterpret_cast<bf16x4*>(dst) = o;
      }
    }
  }
}

template <int XM, int WM, int EPI, int NB, bool EARLY>
hipError_t launch_gemm_tiles(GemmParams p, int t_begin, int t_end, hipStream_t stream) {
  p.t_begin = t_begin;
  p.ntx = (t_end - t_begin + 32 * NB - 1) / (32 * NB);
  const int64_t tiles = (int64_t)p.ntx * p.nfy;
  if (tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)(8 * ((tiles + 7) / 8)));
  hipLaunchKernelGGL((gemm_kernel<XM, WM, EPI, NB, EARLY>), grid, dim3(NB < 8 ? 2 * kGemmThreads : kGemmThreads),
                     0, stream, p);
  return hipGetLastError();
}

template <int XM, int WM, int EPI>
hipError_t launch_gemm(GemmParams p, hipStream_t stream) {
  const int per_wg = WM == kWGateUp ? kBF / 2 : kBF;
  p.nfy = (p.F + per_wg - 1) / per_wg;
  const GemmSplit sp = gemm_split(p.T, p.nfy);
  const int mid = sp.nb == 8 ? p.T : 256 * sp.full;
  hipError_t e = hipSuccess;
  if (p.K >= 8192) e = launch_gemm_tiles<XM, WM, EPI, 8, true>(p, 0, mid, stream);
  else e = launch_gemm_tiles<XM, WM, EPI, 8, false>(p, 0, mid, stream);
  if (e != hipSuccess) return e;
  switch (sp.nb) {
    case 4: return launch_gemm_tiles<XM, WM, EPI, 4, false>(p, mid, p.T, stream);
    case 3: return launch_gemm_tiles<XM, WM, EPI, 3, false>(p, mid, p.T, stream);
    case 2: return launch_gemm_tiles<XM, WM, EPI, 2, false>(p, mid, p.T, stream);
    default: return hipSuccess;
  }
}

}  // namespace
}  // namespace apb

#endif  // APB_GEMM_H_
